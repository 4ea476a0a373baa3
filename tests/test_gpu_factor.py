"""The factorisation at the edges of its tiles and pivot blocks, through the
local solves it feeds: one subdomain, so the apply is the whole grid's inverse
and the oracle's direct solve is its reference."""
import numpy as np
import pytest

from oracle import oras as ooras
from paper_2110_15113_amd import workloads as wl

from gpu_util import (EPS32, FP32_BOX, FP64_BOX, box_err, need_gpu, oracle_fields, rand_field,
                      say, setup, to_dev)

pytestmark = pytest.mark.gpu


# plane sizes around whole tiles of 32 rows, pivot blocks of 2 (complex128)
# and 4 (complex64) tiles, and 16-row blocks inside them
@pytest.mark.parametrize("nx,ny", [(5, 3), (4, 4), (16, 2), (11, 3), (8, 8), (13, 5), (16, 6),
                                   (97, 1 + 1), (16, 8), (43, 3), (9, 17), (32, 8), (29, 9)])
def test_factor_edges(nx, ny):
    need_gpu()
    say(f"factor plane {nx}x{ny}")
    nz = 6
    # the grid needs 3 nodes per axis: thinner planes come from two parts along y
    parts = (1, 1, 1) if ny >= 3 else (1, 2, 1)
    n = (nx, ny if ny >= 3 else 4, nz)
    w = wl.small_random(n, npml=1, q=50.0, seed=71)
    x = rand_field((w.nz, w.ny, w.nx), 2, 72)
    ref = ooras.ORAS(oracle_fields(w), parts, 0).apply(x)
    for prec, bar in ((2, FP64_BOX), (1, FP32_BOX)):
        S = setup(w, prec=prec, parts=parts, overlap=0)
        y = S.apply_M(to_dev(x, S)).cpu().numpy()
        e = box_err(y, ref, parts, 0)
        say(f"  prec {prec}: {e:.2e}")
        assert np.isfinite(e) and e < bar


# boxes of one tile and of five: pivot panels are packed into the scratch plane
# of P x P entries a subdomain has for T, however few tiles a plane holds
@pytest.mark.parametrize("n,parts", [((32, 32, 32), (16, 16, 16)), ((96, 96, 16), (8, 8, 4))])
@pytest.mark.parametrize("prec", [1, 2])
def test_factor_memory(n, parts, prec):
    need_gpu()
    import torch
    w = wl.small_random(n, npml=1, q=50.0, seed=73)
    S = setup(w, prec=prec)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    S.factor(parts, 0, prec)
    used = before - torch.cuda.mem_get_info()[0]
    box = [n[a] // parts[a] for a in range(3)]
    P = -(-box[0] * box[1] // 32) * 32
    entry = 8 if prec == 1 else 16
    sub = (box[2] + 1) * P * P + 27 * box[0] * box[1] * box[2]    # factors, scratch, couplings
    nsub = parts[0] * parts[1] * parts[2]
    say(f"factor memory {n} {parts} prec {prec}: {used} of {nsub * sub * entry}")
    # descriptors and statistics: well below 1 KB a subdomain, 2 MB pages
    assert used <= nsub * (sub * entry + 1024) + (16 << 20)


@pytest.mark.parametrize("n,parts,ov", [((11, 58, 3), (5, 3, 1), 8), ((3, 203, 11), (1, 1, 1), 2)])
def test_factor_near_small_pivots(n, parts, ov):
    """Thin boxes of forty rough models, whose pivots go down to r = 1e-3 of
    their plane's largest entry.  Elimination without row exchanges makes backward
    errors of eps / r, in each of the 2 s_z plane products of a local solve;
    block rows and columns that belong to different matrices (a diagonal block's
    inverse that is not symmetric) leave eps / r^2."""
    need_gpu()
    import torch
    from oracle import operator as op
    from paper_2110_15113_amd import oras
    nx, ny, nz = n
    omega, h = 2 * np.pi * 6.0, 20.0
    x = rand_field((nz, ny, nx), 1, 90)
    S = oras.Solver(0)
    worst = 0.0
    for seed in range(40):
        g = torch.Generator().manual_seed(seed)
        vel = 1500 + 3000 * torch.rand((nz, ny, nx), generator=g, dtype=torch.float64)
        ref = ooras.ORAS(op.make_fields(vel.numpy(), None, omega, h, 1), parts, ov).apply(x)
        S.assemble(vel.to(S.device), h, 1, omega, prec=1)
        S.factor(parts, ov, 1)
        r = S.factor_stats()[0]
        y = S.apply_M(to_dev(x, S)).cpu().numpy()
        e = float(np.linalg.norm(y - ref) / np.linalg.norm(ref))
        worst = max(worst, e * r / (2 * nz * EPS32))
        assert e < 2 * nz * EPS32 / r, (seed, r, e)
    say(f"small pivots {n}: at most {worst:.2f} of the bar")


@pytest.mark.parametrize("n,npml,seed", [((18, 23, 37), 0, 33), ((18, 23, 37), 0, 39),
                                         ((18, 23, 37), 0, 23), ((26, 44, 3), 1, 49)])
def test_factor_after_a_nearly_singular_plane(n, npml, seed):
    """One box of a rough model that is well conditioned as a whole (a complex64
    solve with row exchanges within the planes errs by 2e-6, 4e-7, 4e-7 and 2e-5)
    but not every plane, so that the next one begins as a large multiple s of a
    rank-one matrix.  Elimination row by row leaves eps s, which the eps / r of the
    test above covers; products with the inverses of 16 x 16 blocks leave eps s^2."""
    need_gpu()
    import torch
    from oracle import operator as op
    from paper_2110_15113_amd import oras
    nx, ny, nz = n
    omega, h = 2 * np.pi * 6.0, 20.0
    g = torch.Generator().manual_seed(seed)
    vel = 1500 + 3000 * torch.rand((nz, ny, nx), generator=g, dtype=torch.float64)
    x = torch.randn((3, nz, ny, nx), generator=g, dtype=torch.complex128)
    M = ooras.ORAS(op.make_fields(vel.numpy(), None, omega, h, npml), (1, 1, 1), 0)
    S = oras.Solver(0)
    S.assemble(vel.to(S.device), h, npml, omega, prec=1)
    S.factor((1, 1, 1), 0, 1)
    r = S.factor_stats()[0]
    Y = S.apply_M(x.to(S.device)).cpu().numpy()
    for b in range(3):
        ref = M.apply(x[b].numpy())
        e = float(np.linalg.norm(Y[b] - ref) / np.linalg.norm(ref))
        say(f"near-singular plane {n} seed {seed}: r {r:.1e}, {e * r / (2 * nz * EPS32):.2f} of the bar")
        assert e < 2 * nz * EPS32 / r, (r, e)
