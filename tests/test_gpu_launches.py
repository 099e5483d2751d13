"""GPU parity of the forms a step's launches take: level substeps that share
a launch, and the rules that choose a launch's shape.  FP64 results equal the
oracle's bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_2402_04606_amd as P
    P.lib()
    return P, oracle


def equal_levels(g, o, wl, c=0):
    for l in range(wl.n_levels):
        for name, a, b in zip(("rho", "ux", "uy"), g.fields(c, l), o.fields(l)):
            assert np.array_equal(a, b, equal_nan=True), (wl.name, l, name)


def nest(m, walls):
    """m nested levels over the centre of a 64^2 domain: the last launch of a
    step holds a substep of every level, with up to three roles each."""
    boxes = [(1, 2, 2, 6, 6), (2, 6, 6, 10, 10), (3, 14, 14, 18, 18), (4, 30, 30, 34, 34), (5, 62, 62, 66, 66)]
    wl = W.tgv(64, tau=0.51, n_levels=m, boxes=boxes[:m - 1], name=f"nest{m}{'w' if walls else ''}")
    return wl.replace(bc=(W.WALL,) * 4, bc_u=((0.0, 0.0),) * 3 + ((0.02, 0.0),)) if walls else wl


@pytest.mark.parametrize("m,walls,remap,tile", [(2, True, 1, 0), (4, False, 0, 1), (6, True, 1, 0), (6, True, 0, 2),
                                                (6, False, 1, 3)])
def test_shared_launches_match_oracle(env, m, walls, remap, tile):
    """6 walled levels give 17 launch entries (7 share the header's load)."""
    P, O = env
    wl = nest(m, walls)
    print(wl.name, remap, tile, flush=True)
    g, o = P.Sim(wl, "f64"), O.OracleSim(wl)
    g.set_option(P.OPT_XCD_REMAP, remap)
    g.set_option(P.OPT_TILE, tile)
    g.step(5)
    g.synchronize()
    o.step(5)
    equal_levels(g, o, wl)


@pytest.mark.parametrize("tile", [0, 3])
def test_solid_blocks_share_the_launch(env, tile):
    P, O = env
    wl = W.cavity_ibb()
    print(wl.name, tile, flush=True)
    g, o = P.Sim(wl, "f64"), O.OracleSim(wl)
    g.set_option(P.OPT_TILE, tile)
    g.step(3)
    g.synchronize()
    o.step(3)
    equal_levels(g, o, wl)
