"""The built level kernels, read back as assembly on the CPU: a lane's store to
LDS is complete before the barrier behind which other waves read it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2402_04606_amd", "libsbt.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of every level_tile_kernel<storage, buffers, solid>."""
    if not (os.path.exists(LIB) and os.path.exists(OBJDUMP)):
        pytest.skip("libsbt.so not built, or no disassembler")
    d = str(tmp_path_factory.mktemp("isa"))
    shutil.copy(LIB, os.path.join(d, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    found = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", f], cwd=d, check=True,
                              capture_output=True, text=True).stdout
        body = None
        for line in text.splitlines():
            if line.startswith("<"):
                m = re.search(r"level_tile_kernelILi(\d)ELi(\d)ELb(\d)E", line)
                body = found.setdefault(tuple(map(int, m.groups())), []) if m else None
            elif body is not None and line.startswith("\t"):
                body.append(line.split("//")[0].strip())
    return found


@pytest.mark.parametrize("storage", range(8))
def test_lds_stores_complete_before_a_barrier(kernels, storage):
    mine = {k: v for k, v in kernels.items() if k[0] == storage}
    assert len(mine) == 4, sorted(kernels)
    seen = 0
    for name, body in mine.items():
        for i, ins in enumerate(body):
            if not ins.startswith("ds_write"):
                continue
            waited = False
            for nxt in body[i + 1:i + 400]:
                if nxt.startswith(("s_branch", "s_endpgm", "s_setpc")):
                    break
                waited |= nxt.startswith("s_waitcnt") and "lgkmcnt(0)" in nxt
                if nxt.startswith("s_barrier"):
                    assert waited, (name, i, ins)
                    seen += 1
                    break
    assert seen >= 4
