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


def ring(n, r, centre=(64.0, 64.0), nx=128, ny=128):
    """A fixed ring of n markers of radius r in a uniform stream."""
    wl = W.cylinder(nx, ny, D=2 * r, centre=centre, n_markers=n, perturb=False)
    return wl.replace(name=f"ring{n}_r{r}")


@pytest.mark.parametrize("wl", [
    ring(6, 4.0),                               # waves without markers
    ring(128, 20.0),                            # two lanes per marker: a full wave of pairs
    ring(512, 60.0), ring(513, 60.0),           # the last body with two lanes per marker, the first with one
    ring(200, 1.5),                             # more than 63 markers over a cell: the last count bin
    ring(300, 95.0, (160.0, 160.0), 320, 320),  # a window beyond LDS, more than 2048 stencil cells
], ids=lambda w: w.name)
def test_forcing_plans_match_oracle(env, wl):
    P, O = env
    print(wl.name, flush=True)
    g, o = P.Sim(wl, "f64"), O.OracleSim(wl)
    g.step(4)
    g.synchronize()
    o.step(4)
    equal_levels(g, o, wl)
    for a, b in zip(g.force_history(), o.force_history()):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("m", [2, 4])
def test_plans_follow_the_state(env, m):
    """Plans built ahead of their substeps: after a checkpoint is restored,
    and around a persistent step (which builds its own), the run goes on as
    an unbroken one; so does a fixed body beside a moving one."""
    P, O = env
    wls = [W.small_refined_flap(m=m), ring(40, 8.0).replace(name="ring"), W.small_pitch_up(m=min(m, 3))]
    print(m, flush=True)

    def history(g):
        g.synchronize()
        return [np.array(g.force_history(c)) for c in range(len(wls))]

    ref = P.Sim(wls, "f64")
    ref.step(9)
    g = P.Sim(wls, "f64")
    g.step(3)
    state = g.read_state()
    g.step(2)
    g.write_state(state)
    g.step(1)
    g.set_option(P.OPT_PERSISTENT, 1)
    g.step(2)
    g.set_option(P.OPT_PERSISTENT, 0)
    g.step(1)
    g.set_option(P.OPT_GRAPH, 0)
    g.step(2)
    for a, b in zip(history(g), history(ref)):
        assert np.array_equal(a, b)


def test_many_bodies_match_one(env):
    """130 bodies leave no CUs for plans beside the loops: a launch of their
    own builds them."""
    P, O = env
    wl = W.small_refined_flap(m=2)
    print(wl.name, flush=True)
    one, many = P.Sim(wl, "f32", history_cap=64), P.Sim([wl] * 130, "f32", history_cap=64)
    one.step(5)
    many.step(5)
    want = np.array(one.force_history(0, 64))
    assert np.isfinite(want).all() and want.shape[1] > 0
    for c in (0, 64, 129):
        assert np.array_equal(np.array(many.force_history(c, 64)), want)


def marker_box(n, moving):
    """n markers on a small sphere (or a pitching, plunging ellipsoid)."""
    if moving:
        return W.flapping_ellipsoid3(n=32, chord=12.0, n_markers=n)
    return W.ibm_sphere3(n=24, r=4.0, n_markers=n, g=1e-6)


@pytest.mark.parametrize("n,moving", [(1, False), (16, True), (17, False), (65, True), (1024, False), (1025, True)])
def test_forcing_loop3_matches_oracle(env, n, moving):
    """Marker counts around a workgroup's 16, a wave's 64 and a block's 1024."""
    P, O = env
    wl = marker_box(n, moving)
    print(wl.name, n, flush=True)
    g, o = P.Sim3(wl, "f64"), O.Oracle3Sim(wl)
    for _ in range(2):
        g.step(2)
        g.synchronize()
        o.step(2)
        assert np.array_equal(g.body_force(), o.body_force())
    for a, b in zip(g.fields(), o.fields()):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("sizes,mrt", [(((16, 16),), False), (((48, 32), (16, 80)), True), (((272, 256),), False),
                                       (((512, 528),), True)])
def test_steps_that_share_a_launch(env, storage, sizes, mrt):
    """Calls of many steps against single steps, bit for bit, state included:
    a block that is its own neighbour, a batch, 256 blocks and more (four or
    two steps a launch), a body force, every remainder of a call."""
    P, O = env
    wls = []
    for c, (nx, ny) in enumerate(sizes):
        wl = W.tgv(64, tau=0.6 + 0.1 * c, u0=0.03)
        wls.append(wl.replace(nx0=nx, ny0=ny, fext=(1e-5, -2e-5), collision=W.COLL_MRT if mrt else W.COLL_BGK))
    print(sizes, storage, mrt, flush=True)
    one, many = P.Sim(wls, storage), P.Sim(wls, storage)
    for n in (5, 6, 7, 8, 9, 13, 1, 26):
        for _ in range(n):
            one.step(1)
        many.step(n)
        many.synchronize()
        assert np.array_equal(one.read_state(), many.read_state()), n
    for c in range(len(wls)):
        for a, b in zip(one.fields(c, 0), many.fields(c, 0)):
            assert np.array_equal(a, b)
    if storage == "f64" and not mrt and sizes[0][0] < 100:
        o = O.OracleSim(wls[0])
        o.step(75)
        equal_levels(many, o, wls[0])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("m,mrt,remap", [(1, False, 1), (1, True, 0), (2, True, 1), (4, False, 1), (4, True, 0)])
def test_forcing_loops_that_share_a_launch(env, storage, m, mrt, remap):
    """Forcing loops and the collisions that wait for them in one launch
    against launches of their own (which the profiler times), bit for bit:
    fixed and moving bodies, plans beside them, every part of a level, odd
    and even counts of substeps, replayed and eager."""
    P, O = env
    wls = [ring(126, 20.0), ring(40, 8.0, (30.0, 90.0))]
    if m > 1:
        wls += [W.small_refined_flap(m=m), W.small_pitch_up(m=min(m, 3))]
    wls = [w.replace(collision=W.COLL_MRT if mrt else W.COLL_BGK) for w in wls]
    print(storage, m, mrt, remap, flush=True)
    # one entry of force history: all of the state is written by the first step
    apart, shared = P.Sim(wls, storage, history_cap=1), P.Sim(wls, storage, history_cap=1)
    for g in (apart, shared):
        g.set_option(P.OPT_XCD_REMAP, remap)
    for n in (1, 2, 7, 4, 3):
        apart.profile(n)
        shared.step(n)
        shared.synchronize()
        assert np.array_equal(apart.read_state(), shared.read_state()), n
        shared.set_option(P.OPT_GRAPH, n != 7)
    for c in range(len(wls)):
        a, b = np.array(apart.force_history(c, 1)), np.array(shared.force_history(c, 1))
        assert a.shape == b.shape and a.size and np.array_equal(a, b), c


@pytest.mark.parametrize("bodies_share", [True, False])
def test_bodies_far_from_the_origin(env, bodies_share):
    """A ring under six levels of a periodic plane, moved to finest cells
    beyond 32768 in y and beyond 65536 in x by whole level-0 blocks: marker
    positions are exact in both places, so every bit of the run moves along."""
    P, O = env
    m, r = 6, 8.0

    def placed(kx, ky):
        wl = nest(m, False)
        ring40 = ring(40, r).body
        xb, yb = (np.round(np.asarray(v) * 4096.0) / 4096.0 for v in (ring40.xb, ring40.yb))
        boxes = [(l, x0 + (kx << l), y0 + (ky << l), x1 + (kx << l), y1 + (ky << l)) for l, x0, y0, x1, y1 in wl.boxes]
        p = [1024.25 + 512 * kx, 1024.25 + 512 * ky] + [0.0] * 14
        return wl.replace(nx0=16 * 133, ny0=16 * 69, boxes=boxes, init=W.uniform_init(1.0, 0.05, 0.01),
                          body=W.Body(W.BODY_FIXED, xb, yb, ring40.ds, p))

    def run(kx, ky):
        print(kx, ky, bodies_share, flush=True)
        g = P.Sim(placed(kx, ky), "f64")
        if bodies_share:
            g.step(2)
        else:
            g.profile(2)
        g.synchronize()
        return np.array(g.force_history(0)), [np.roll(f, (-16 * ky, -16 * kx), (0, 1)) for f in g.fields(0, 0)]

    h0, f0 = run(0, 0)
    assert np.isfinite(h0).all() and np.abs(h0).max() > 0
    for at in ((0, 65), (129, 0), (129, 65)):
        h, f = run(*at)
        assert np.array_equal(h, h0), at
        assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(f, f0)), at


@pytest.mark.parametrize("m", [5, 6])
def test_plans_behind_a_single_loop(env, m):
    """One moving body on 5 and 6 levels: 8 and 16 plans beside one loop, more
    than the first eight workgroups of a launch take."""
    P, O = env
    wl = W.small_refined_flap(m=m)
    print(wl.name, flush=True)
    apart, shared = P.Sim(wl, "f32", history_cap=1), P.Sim(wl, "f32", history_cap=1)
    for n in (1, 3, 4):
        apart.profile(n)
        shared.step(n)
        shared.synchronize()
        assert np.array_equal(apart.read_state(), shared.read_state()), n


def test_a_wait_that_gives_up_is_reported(env):
    """One poll per wait (set from the host): the launch ends normally,
    synchronize reports it once, and after write_state with the default limit
    the context steps as one that never gave up."""
    P, O = env
    wl = ring(126, 20.0)
    print(wl.name, flush=True)
    # one entry of force history: all of the state is written by the first step
    g, ref = P.Sim(wl, "f64", history_cap=1), P.Sim(wl, "f64", history_cap=1)
    for s in (g, ref):
        s.step(5)
        s.synchronize()
    state = g.read_state()
    g.set_option(P.OPT_BARRIER_SPINS, 1)
    g.step(2)
    with pytest.raises(P.SbtError) as e:
        g.synchronize()
    assert e.value.code == -3
    g.synchronize()
    g.set_option(P.OPT_BARRIER_SPINS, 0)
    g.write_state(state)
    for s in (g, ref):
        s.step(6)
        s.synchronize()
    assert np.array_equal(g.read_state(), ref.read_state())


def test_contexts_on_two_streams(env):
    """Two contexts, each with several bodies and more level workgroups than
    the chip holds at once, step at the same time on streams of their own: the
    blocks of one that wait never keep the other's loops from running."""
    import torch
    P, O = env
    a = [ring(126, 20.0, (150.0, 256.0), 1024, 512), ring(40, 8.0, (30.0, 90.0))]
    b = [W.small_refined_flap(m=4), ring(200, 24.0, (200.0, 256.0), 1024, 512)]
    refs = [P.Sim(w, "f32", history_cap=1) for w in (a, b)]
    for g in refs:
        g.step(120)
        g.synchronize()
    both = [P.Sim(w, "f32", history_cap=1, stream=torch.cuda.Stream()) for w in (a, b)]
    for n in range(30):
        for g in both:
            g.step(4)
    print("issued", flush=True)
    for g, ref in zip(both, refs):
        g.synchronize()
        assert np.array_equal(g.read_state(), ref.read_state())


def test_autotune_times_the_launches_it_chooses_for(env, tmp_path):
    """Its trials run one step per launch, also on a level where a long call
    runs several: only then do the candidates differ."""
    import torch
    P, O = env
    g = P.Sim(W.tgv(64), "f32")
    print("tgv64", flush=True)

    def kernels(f):
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
            f()
            g.synchronize()
        return " ".join(e.name for e in prof.events())

    names = kernels(lambda: g.step(24))
    assert "multi_step_kernel" in names
    before = g.read_state()
    names = kernels(lambda: g.autotune(steps=24, cache_path=str(tmp_path / "tune.json")))
    assert "level_tile_kernel" in names and "multi_step_kernel" not in names
    assert np.array_equal(g.read_state(), before)
    assert "multi_step_kernel" in kernels(lambda: g.step(24))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "bf16s"])
@pytest.mark.parametrize("lattice", [19, 27])
def test_one_level_forest_matches_oracle(env, storage, lattice):
    """A forest without refinement is a schedule of one launch a step."""
    from test_gpu_forest3d import _compare
    P, O = env
    wl = W.vortex3f(n0=32, m=1, boxes=(), lattice=lattice).replace(nx0=32, ny0=48, nz0=40)
    print(storage, lattice, flush=True)
    g, o = P.Sim3F(wl, storage), O.Oracle3FSim(wl)
    g.step(6)
    g.synchronize()
    o.step(6)
    _compare(g, o, wl, storage)


@pytest.mark.parametrize("size,box", [
    ((136, 128, 72), (0, 0, 0, 136, 128, 72)),     # whole planes
    ((136, 128, 72), (3, 5, 6, 131, 121, 65)),     # off the block faces
    ((400, 384, 24), (1, 0, 5, 399, 384, 19)),     # whole planes, fewer than a block's
    ((528, 256, 24), (1, 0, 4, 527, 255, 19)),     # rows of eight planes
    ((528, 256, 24), (0, 3, 7, 528, 250, 5)),      # fewer planes than a block
    ((16392, 8, 16), (5, 1, 3, 16387, 7, 12)),     # cells of eight rows
], ids=str)
def test_boxes_larger_than_the_staging_area(env, size, box):
    """A readout cut into parts against readouts that fit in one."""
    P, O = env
    wl = W.vortex3f(n0=32, m=1, boxes=()).replace(nx0=size[0], ny0=size[1], nz0=size[2])
    print(size, box, flush=True)
    g = P.Sim3F(wl, "f32")
    g.step(2)
    whole = g.fields(0, box)
    x0, y0, z0, nx, ny, nz = box
    for z in range(0, nz, 3):
        for x in range(0, nx, 2999):
            dx, dz = min(2999, nx - x), min(3, nz - z)
            part = g.fields(0, (x0 + x, y0, z0 + z, dx, ny, dz))
            for a, b in zip(whole, part):
                assert np.isfinite(b).all() and np.array_equal(a[z:z + dz, :, x:x + dx], b), (x, z)


@pytest.mark.parametrize("storage", ["f64", "f16s"])
@pytest.mark.parametrize("wl", [ring(512, 40.0), ring(256, 40.0), W.flapping_ellipse(n_markers=402)],
                         ids=["ring512", "ring256", "wing402"])
def test_long_forcing_loops_that_share_a_launch(env, wl, storage):
    """Bodies of up to 512 markers on an arc of at most 256 cells, the largest
    that share a launch, against launches of their own."""
    P, O = env
    print(wl.name, storage, flush=True)
    apart, shared = P.Sim(wl, storage, history_cap=1), P.Sim(wl, storage, history_cap=1)
    for n in (1, 4):
        apart.profile(n)
        shared.step(n)
        shared.synchronize()
        assert np.array_equal(apart.read_state(), shared.read_state()), n


@pytest.mark.parametrize("make", [lambda: W.tgv(64), lambda: nest(1, True), lambda: nest(3, False), lambda: ring(40, 8.0),
                                  lambda: W.small_refined_flap(m=2)], ids=["plane", "walls", "nest", "ring", "flap"])
def test_graphs_are_captured_at_the_first_step(env, make):
    """All graphs that a run can reach: no later step captures one."""
    import torch
    P, O = env
    wl = make()
    print(wl.name, flush=True)
    g = P.Sim(wl, "f32")

    def captures(n):
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
            g.step(n)
            g.synchronize()
        return sum(e.name == "hipGraphInstantiate" for e in prof.events())

    assert captures(1) == 6
    assert [captures(n) for n in (1, 1, 3, 2, 4, 5, 1)] == [0] * 7


@pytest.mark.parametrize("n0,boxes", [(32, ((1, 2, 2, 2, 6, 6, 6),)),               # level 1 of 2^18 cells, an eighth owned
                                      (40, ((1, 1, 1, 1, 5, 9, 9),)),               # 512000 cells, a third
                                      (48, ((1, 2, 2, 2, 6, 6, 6),))], ids=str)     # more than 2^19 cells
def test_readouts_of_a_level_owned_in_part(env, n0, boxes):
    """Boxes with NaN around and inside the owned cells, in and out of the part
    that the level's blocks span, against the oracle."""
    P, O = env
    wl = W.vortex3f(n0=n0, boxes=boxes)
    print(n0, boxes, flush=True)
    g, o = P.Sim3F(wl, "f64"), O.Oracle3FSim(wl)
    g.step(2)
    o.step(2)
    n = 2 * n0
    for l, box in ((1, (0, 0, 0, n, n, n)), (1, (5, 3, 7, n - 6, n - 9, n - 11)), (1, (0, 0, 0, 7, 6, 5)),
                   (1, (n - 20, 0, 0, 20, n, n)), (1, (17, 18, 19, 9, 3, 20)), (0, (0, 0, 0, n0, n0, n0)), (0, (9, 9, 9, 6, 5, 4))):
        want = o.fields(l)
        x, y, z, nx, ny, nz = box
        for a, b in zip(g.fields(l, box), want):
            assert np.array_equal(a, b[z:z + nz, y:y + ny, x:x + nx], equal_nan=True), (l, box)
