"""Data that lanes of one wave hand to each other through LDS without a barrier
of the work-group: in the compiled intermediate code a fence of the wave stands
between one lane's stores and another lane's accesses of the same bytes, so that
no pass of the compiler may move them past each other."""
import os
import re
import subprocess

import pytest


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    from paper_2110_15113_amd import build
    out = str(tmp_path_factory.mktemp("ir") / "k_factor.ll")
    cmd = [build._hipcc(), "-xhip", *build.COMMON, "--cuda-device-only", "-S", "-emit-llvm",
           os.path.join(build.CSRC, "k_factor.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return {m.group(1): m.group(0)
                for m in re.finditer(r"^define[^\n]*?@(\w+)\(.*?^}", f.read(), re.S | re.M)}


def order(body):
    """LDS stores (S) and loads (L) and the wave's fences (F), in order."""
    found = re.findall(r"(store) [^\n]*addrspace\(3\)|(load) [^\n]*addrspace\(3\)|"
                       r'(fence) syncscope\("wavefront"\)', body)
    return "".join("S" if s else "L" if l else "F" for s, l, _ in found)


def test_panel_tile_through_lds(kernels):
    body, = [v for k, v in kernels.items() if "gj_panel_kernelIf" in k]
    # up to the work-group's barrier: the tile is stored, read by columns, and
    # stored again in its split form over the same bytes
    seq = order(body.split('fence syncscope("workgroup")')[0])
    assert re.fullmatch("S+F+L+F+S+", seq), seq


@pytest.mark.parametrize("real", ["f", "d"])
def test_pivot_block_through_lds(kernels, real):
    body, = [v for k, v in kernels.items() if "gj_diag_kernelI" + real in k]
    # the wave that runs ahead: its product's stores, then the loads of the
    # inverse, whose first pivot is a lane read
    seq = order(body.split("s.setprio(i16 3)")[1].split("amdgcn.readlane")[0])
    assert re.fullmatch("L+S+F+L+", seq), seq
