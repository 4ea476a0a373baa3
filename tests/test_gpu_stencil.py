"""Parity of the matrix-free 27-point apply with the oracle's assembled rows,
element by element (paper sec. 2.3, FDFD stencil).

The apply forms each row's coefficients from node fields and the 1D PML
profiles inside the kernel, with a reduced form on tiles the PML does not
reach.  The grids below are sized so that both kinds of tile run in one apply (8 x 8
x 16 tiles: with npml = 3 the nodes 4 .. n - 5 use only unit profile values,
so the first grid has PML-free tiles at planes 16 .. 31), with ragged tiles
on every axis, and one grid has no PML at all.  The chunk widths differ by
kind (32 right-hand sides on PML tiles, 16 elsewhere in single precision), so
the right-hand-side counts cover full and partial chunks of both.  The bar is per
entry, relative to sum_e |c_e| |x_e| of that row (the size of the terms the
entry sums), so a wrong coupling in one row or one tile fails on its own.
"""
import numpy as np
import pytest

from oracle import operator as op
from paper_2110_15113_amd import workloads as wl

from gpu_util import EPS32, need_gpu, oracle_fields, rand_field, say, setup, to_dev

pytestmark = pytest.mark.gpu

FP64_ROW = 1e-12
# x, the node fields and the coefficient arithmetic in single precision: a
# few roundings per term and 27 terms per row
FP32_ROW = 32 * EPS32

CASES = [
    dict(n=(40, 36, 38), npml=3, q=80.0, nrhs=1, seed=31),    # PML and interior tiles
    dict(n=(37, 20, 19), npml=2, q=None, nrhs=13, seed=32),   # ragged tiles, 2 chunks
    dict(n=(21, 18, 11), npml=0, q=50.0, nrhs=40, seed=33),   # no PML: interior tiles only
    dict(n=(33, 17, 21), npml=2, q=70.0, nrhs=50, seed=37),   # chunks of 32, 16 and 8 RHS
    dict(n=(18, 17, 9), npml=2, q=None, nrhs=256, seed=38),   # the widest block
]


def _row_err(got, ref, scale):
    return float((np.abs(got - ref) / scale).max())


@pytest.mark.parametrize("case", CASES)
def test_matrix_free_apply_matches_oracle_rows(case):
    need_gpu()
    w = wl.small_random(case["n"], npml=case["npml"], q=case["q"], seed=case["seed"])
    say(f"matrix-free apply {w.name} nrhs={case['nrhs']}")
    S = setup(w, prec=1)          # single-precision stencil (plus the FP64 one)
    x = rand_field((w.nz, w.ny, w.nx), case["nrhs"], case["seed"] + 100)
    C = op.row_coeffs(oracle_fields(w))
    ref = op.apply_coeffs(C, x)
    scale = op.apply_coeffs(np.abs(C), np.abs(x)).real
    assert scale.min() > 0
    y128 = S.apply_A(to_dev(x, S), prec=2).cpu().numpy()
    e128 = _row_err(y128, ref, scale)
    y64 = S.apply_A(to_dev(x, S), prec=1).cpu().numpy()
    e64 = _row_err(y64, ref, scale)
    say(f"  row error: FP64 {e128:.2e}, FP32 {e64:.2e}")
    assert e128 < FP64_ROW
    assert e64 < FP32_ROW


def test_matrix_free_apply_after_set_m():
    """A new squared slowness rebuilds the node fields the apply reads."""
    need_gpu()
    import torch
    w = wl.small_random((34, 19, 18), npml=2, q=60.0, seed=34)
    S = setup(w, prec=1)
    rng = np.random.default_rng(35)
    m = (1.0 / w.vel ** 2) * (1.0 + 0.2 * rng.random(w.vel.shape))
    S.set_m(torch.as_tensor(m, device=S.device))
    x = rand_field((w.nz, w.ny, w.nx), 3, 36)
    F = op.make_fields(w.vel, w.Q, w.omega, w.h, w.npml, m=m)   # weights kept from vel
    C = op.row_coeffs(F)
    ref = op.apply_coeffs(C, x)
    scale = op.apply_coeffs(np.abs(C), np.abs(x)).real
    y128 = S.apply_A(to_dev(x, S), prec=2).cpu().numpy()
    y64 = S.apply_A(to_dev(x, S), prec=1).cpu().numpy()
    assert _row_err(y128, ref, scale) < FP64_ROW
    assert _row_err(y64, ref, scale) < FP32_ROW


# grids whose applies run tiles of 2, 4, 8 and 16 planes (8 x 8 columns, the
# tallest with 512 work items in single precision, 400 in double): 25 x 2,
# 25 x 11 x 2, 36 x 5 x 3 and 64 x 3 x 3 tiles times chunks of 16
@pytest.mark.parametrize("n,nrhs", [((33, 34, 3), 1), ((33, 34, 41), 17), ((41, 42, 37), 33),
                                    ((57, 58, 33), 35)])
def test_apply_of_caller_arrays(n, nrhs):
    """Every tile height against the oracle's rows; an output that overlaps
    the input takes the staged path and agrees with the direct one."""
    need_gpu()
    w = wl.small_random(n, npml=1, q=70.0, seed=61)
    S = setup(w, prec=1)
    x = rand_field((w.nz, w.ny, w.nx), nrhs, 62)
    C = op.row_coeffs(oracle_fields(w))
    ref = op.apply_coeffs(C, x)
    scale = op.apply_coeffs(np.abs(C), np.abs(x)).real
    for prec, bar in ((2, FP64_ROW), (1, FP32_ROW)):
        xd = to_dev(x, S)
        y = S.apply_A(xd, prec=prec)
        assert _row_err(y.cpu().numpy(), ref, scale) < bar
        if nrhs * w.nx * w.ny * w.nz * 40 < 5e7:
            S.apply_A_noalloc(xd, xd, prec=prec)      # in place
            assert _row_err(xd.cpu().numpy(), ref, scale) < bar


# 64 x 3 tiles, some of them PML-free, in 3 and in 4 chunks of 16: below and at
# the 768 work items from which PML-free tiles have a launch of their own in
# double precision (the 24 columns: one chunk of 16 and one of 8)
@pytest.mark.parametrize("nrhs", [24, 48, 64])
def test_apply_in_one_launch_or_two(nrhs):
    need_gpu()
    w = wl.small_random((57, 58, 33), npml=4, q=70.0, seed=63)
    S = setup(w, prec=1)
    x = rand_field((w.nz, w.ny, w.nx), nrhs, 64)
    C = op.row_coeffs(oracle_fields(w))
    ref = op.apply_coeffs(C, x)
    scale = op.apply_coeffs(np.abs(C), np.abs(x)).real
    for prec, bar in ((2, FP64_ROW), (1, FP32_ROW)):
        y = S.apply_A(to_dev(x, S), prec=prec)
        assert _row_err(y.cpu().numpy(), ref, scale) < bar


# 33 and 48 columns: tiles of 16 planes, as 64 (lower tiles are PML-free more often)
@pytest.mark.parametrize("nrhs", [33, 48])
def test_fp32_apply_does_not_depend_on_the_block(nrhs):
    """A column's single-precision result is bitwise the one it has in a block
    of 64: small calls form the couplings no less exactly than large ones."""
    need_gpu()
    w = wl.small_random((57, 58, 33), npml=4, q=70.0, seed=65)
    S = setup(w, prec=1)
    x = to_dev(rand_field((w.nz, w.ny, w.nx), 64, 66), S)
    big = S.apply_A(x, prec=1)
    assert bool((S.apply_A(x[:nrhs].contiguous(), prec=1) == big[:nrhs]).all())


# y in the place of x, a part of a field above it and a part of a field below
# it; the grids and columns of every tile height
@pytest.mark.parametrize("n,nrhs", [((33, 34, 3), 1), ((33, 34, 41), 17), ((41, 42, 37), 33)])
@pytest.mark.parametrize("prec", [1, 2])
def test_apply_of_overlapping_arrays(n, nrhs, prec):
    """Through the C ABI, which alone takes overlapping arrays: x is read in
    full before y is written, with the values of separate arrays bit for bit."""
    need_gpu()
    import torch
    from paper_2110_15113_amd import oras
    w = wl.small_random(n, npml=1, q=70.0, seed=67)
    S = setup(w, prec=1)
    x = to_dev(rand_field((w.nz, w.ny, w.nx), nrhs, 68), S)
    ref = S.apply_A(x, prec=prec)
    count, part = x.numel(), x[0].numel() // 2 + 1
    calls = [oras.lib().oras_apply_A]
    if count * 48 < oras.lib().oras_noalloc_scratch_bytes():
        calls.append(oras.lib().oras_apply_A_noalloc)
    for call in calls:
        for shift in (0, part, -part):
            buf = torch.full((count + 2 * part,), float("nan"), dtype=torch.complex128,
                             device=S.device)
            xs, ys = buf[part:part + count], buf[part + shift:part + shift + count]
            xs.copy_(x.view(-1))
            S._check(call(S._ctx, oras._ptr(xs), oras._ptr(ys), nrhs, prec))
            assert torch.equal(ys, ref.view(-1)), (call.__name__, shift)
