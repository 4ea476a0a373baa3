"""Block low-rank plane inverses (sec. 3: BLR local factors with threshold
eps_BLR; Table 4) on the GPU against the oracle's BLR local solves."""
import numpy as np
import pytest
import torch

from oracle import blr as oblr, direct, operator as op, oras as ooras
from paper_2110_15113_amd import workloads as wl

from gpu_util import (BLR32_BOX, FP32_BOX, FP64_BOX, box_err, need_gpu, oracle_fields,
                      rand_field, rel, say, setup, to_dev)

pytestmark = pytest.mark.gpu

CASES = [
    dict(n=(18, 16, 14), parts=(2, 2, 1), ov=2, npml=2, q=60.0, pmax=4, nrhs=3),
    dict(n=(23, 21, 12), parts=(1, 1, 2), ov=2, npml=2, q=None, pmax=8, nrhs=9),
    dict(n=(16, 19, 15), parts=(2, 1, 2), ov=1, npml=2, q=80.0, pmax=5, nrhs=37),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("eps", [1e-3, 1e-5])
def test_blr_fp64_ranks_and_apply_match_oracle(case, eps):
    need_gpu()
    w = wl.small_random(case["n"], npml=case["npml"], q=case["q"], seed=9,
                        parts=case["parts"], overlap=case["ov"])
    say(f"blr fp64 {case} eps={eps}")
    F = oracle_fields(w)
    M = oblr.OrasBLR(F, case["parts"], case["ov"], eps, case["pmax"])
    S = setup(w, prec=2, parts=case["parts"], overlap=case["ov"])
    info = S.compress(eps, case["pmax"])
    assert info["lowrank"] > 0
    mismatch = total = 0
    for j, sol in enumerate(M.solvers):
        for k, plane in enumerate(sol.inv):
            got = S.blr_ranks(j, k)
            mismatch += int(np.sum(got != plane.rank))
            total += got.size
    assert mismatch == 0, (mismatch, total)
    x = rand_field((w.nz, w.ny, w.nx), case["nrhs"], 3)
    ref = M.apply(x)
    got = S.apply_M(to_dev(x, S)).cpu().numpy()
    e = box_err(got, ref, case["parts"], case["ov"])
    say(f"  per-box error {e:.2e}")
    assert rel(got, ref) < 1e-9 and e < FP64_BOX, (rel(got, ref), e)


def test_blr_eps_zero_is_the_dense_apply():
    need_gpu()
    c = CASES[1]
    w = wl.small_random(c["n"], npml=c["npml"], q=c["q"], seed=9, parts=c["parts"],
                        overlap=c["ov"])
    say("blr eps 0")
    x = rand_field((w.nz, w.ny, w.nx), 5, 4)
    S = setup(w, prec=2, parts=c["parts"], overlap=c["ov"])
    dense = S.apply_M(to_dev(x, S)).cpu().numpy()
    S.compress(0.0, 8)
    got = S.apply_M(to_dev(x, S)).cpu().numpy()
    assert rel(got, dense) < 1e-12, rel(got, dense)
    # a new factorisation drops the compressed form
    S.factor(c["parts"], c["ov"], 2)
    again = S.apply_M(to_dev(x, S)).cpu().numpy()
    assert rel(again, dense) < 1e-14


@pytest.mark.parametrize("case", CASES)
def test_blr_fp32_eps_zero_matches_exact_local_solves(case):
    """With eps = 0 every block stays dense, so the complex-FP32 BLR products
    (the expansion kernel over dense patch blocks in patch-major order) must
    reproduce the exact local solves to the FP32 per-box bar."""
    need_gpu()
    w = wl.small_random(case["n"], npml=case["npml"], q=case["q"], seed=9,
                        parts=case["parts"], overlap=case["ov"])
    say(f"blr fp32 eps 0 {case}")
    F = oracle_fields(w)
    Md = ooras.ORAS(F, case["parts"], case["ov"])
    S = setup(w, prec=1, parts=case["parts"], overlap=case["ov"])
    info = S.compress(0.0, case["pmax"])
    assert info["lowrank"] == 0, info
    x = rand_field((w.nz, w.ny, w.nx), case["nrhs"], 6)
    got = S.apply_M(to_dev(x, S)).cpu().numpy()
    e = box_err(got, Md.apply(x), case["parts"], case["ov"])
    say(f"  per-box error vs exact local solves {e:.2e}")
    assert e < FP32_BOX, e


@pytest.mark.parametrize("case", CASES)
def test_blr_fp32_apply_matches_oracle(case):
    need_gpu()
    w = wl.small_random(case["n"], npml=case["npml"], q=case["q"], seed=9,
                        parts=case["parts"], overlap=case["ov"])
    say(f"blr fp32 {case}")
    F = oracle_fields(w)
    eps = 1e-3
    M = oblr.OrasBLR(F, case["parts"], case["ov"], eps, case["pmax"])
    Md = ooras.ORAS(F, case["parts"], case["ov"])
    S = setup(w, prec=1, parts=case["parts"], overlap=case["ov"])
    S.compress(eps, case["pmax"])
    x = rand_field((w.nz, w.ny, w.nx), case["nrhs"], 5)
    ref = M.apply(x)
    got = S.apply_M(to_dev(x, S)).cpu().numpy()
    e = box_err(got, ref, case["parts"], case["ov"])
    ex = box_err(got, Md.apply(x), case["parts"], case["ov"])
    say(f"  per-box error vs oracle BLR {e:.2e}, vs exact local solves {ex:.2e}")
    assert e < BLR32_BOX * eps, e
    # the compression error itself: BLR against the exact local solves
    assert rel(got, Md.apply(x)) < 50 * eps, rel(got, Md.apply(x))
    agree = total = 0
    for j, sol in enumerate(M.solvers):
        for k, plane in enumerate(sol.inv):
            got_r = S.blr_ranks(j, k)
            agree += int(np.sum(np.abs(got_r - plane.rank) <= 1))
            total += got_r.size
    assert agree >= 0.95 * total, (agree, total)


@pytest.mark.parametrize("prec", [1, 2])
def test_blr_solve_config1(prec):
    need_gpu()
    w = wl.config1()
    say(f"blr solve config1 prec={prec}")
    F = oracle_fields(w)
    b = op.point_sources(F, w.sources)
    u = direct.solve(op.assemble(F), F.shape, b)
    its = {}
    for blr in (False, True):
        S = setup(w, prec=prec, parts=w.parts, overlap=w.overlap)
        if blr:
            S.compress(1e-3, 8)
        tol = 1e-6 if prec == 1 else 1e-8
        r = S.solve(to_dev(b, S), tol, restart=w.restart)
        assert bool(r.converged.all())
        x = r.x.cpu().numpy()
        assert rel(x, u) < (1e-4 if prec == 1 else 1e-6), rel(x, u)
        its[blr] = int(r.iters.max())
    assert its[True] <= its[False] + 5, its


def test_blr_with_pml_interfaces_matches_oracle():
    """BLR compression of the plane inverses of PML-interface subdomain
    matrices (sec. 2.2 note on the overlap; sec. 3 BLR), FP64 ranks and
    apply against the oracle."""
    need_gpu()
    c = dict(n=(19, 17, 15), parts=(2, 2, 1), ov=3, npml=2, q=50.0, pmax=6, nrhs=5)
    w = wl.small_random(c["n"], npml=c["npml"], q=c["q"], seed=13, parts=c["parts"],
                        overlap=c["ov"])
    say("blr with pml interfaces")
    F = oracle_fields(w)
    M = oblr.OrasBLR(F, c["parts"], c["ov"], 1e-3, c["pmax"], interface="pml")
    S = setup(w, prec=2, parts=c["parts"], overlap=c["ov"], interface="pml")
    S.compress(1e-3, c["pmax"])
    for j, sol in enumerate(M.solvers):
        for k, plane in enumerate(sol.inv):
            assert np.array_equal(S.blr_ranks(j, k), plane.rank), (j, k)
    x = rand_field((w.nz, w.ny, w.nx), c["nrhs"], 8)
    got = S.apply_M(to_dev(x, S)).cpu().numpy()
    ref = M.apply(x)
    assert rel(got, ref) < 1e-9, rel(got, ref)


def test_refactor_after_compression_drops_the_compressed_form():
    """After compressing, a new factorisation (a finer partition) or a new
    assembly (another frequency) must drop the BLR operands, which describe
    the old subdomains and planes: the apply then equals a fresh context's
    dense apply, and the rank tables are gone."""
    need_gpu()
    from paper_2110_15113_amd import oras
    w = wl.small_random((18, 16, 14), npml=2, q=60.0, seed=9, parts=(2, 2, 1), overlap=2)
    say("refactor after compression")
    x = rand_field((w.nz, w.ny, w.nx), 5, 6)
    S = setup(w, prec=2, parts=(2, 2, 1), overlap=2)
    S.compress(1e-3, 4)
    S.factor((2, 2, 2), 1, 2)                 # more, smaller boxes
    with pytest.raises(oras.OrasError) as e:
        S.blr_ranks(0, 0)
    assert e.value.code == 2
    F = setup(w, prec=2, parts=(2, 2, 2), overlap=1)
    xd = to_dev(x, S)
    assert torch.equal(S.apply_M(xd), F.apply_M(to_dev(x, F)))
    F.close()
    S.compress(1e-3, 4)
    w2 = wl.small_random((18, 16, 14), npml=2, q=60.0, seed=9, freq=6.5, parts=(2, 2, 1),
                         overlap=2)
    vel = torch.as_tensor(w2.vel, device=S.device)
    S.assemble(vel, w2.h, w2.npml, w2.omega, torch.as_tensor(w2.Q, device=S.device), prec=2)
    S.factor((2, 2, 1), 2, 2)
    with pytest.raises(oras.OrasError) as e:
        S.blr_ranks(0, 0)
    assert e.value.code == 2
    F = setup(w2, prec=2, parts=(2, 2, 1), overlap=2)
    assert torch.equal(S.apply_M(xd), F.apply_M(to_dev(x, F)))
    F.close()
    S.close()


@pytest.mark.parametrize("nx,ny", [(16, 16), (26, 10), (24, 24)])
def test_blr_many_segments(nx, ny):
    """Dense blocks of 2 x 2 patches: 64, 65 and 144 operand segments per row
    patch (a wave holds 64 of them at a time)."""
    need_gpu()
    w = wl.small_random((nx, ny, 6), npml=2, q=80.0, seed=15, parts=(1, 1, 1), overlap=1)
    say(f"blr segments {nx}x{ny}")
    S = setup(w, prec=1, parts=(1, 1, 1), overlap=1)
    info = S.compress(0.0, 2)
    assert info["lowrank"] == 0, info
    x = rand_field((w.nz, w.ny, w.nx), 9, 16)
    got = S.apply_M(to_dev(x, S)).cpu().numpy()
    e = box_err(got, ooras.ORAS(oracle_fields(w), (1, 1, 1), 1).apply(x), (1, 1, 1), 1)
    say(f"  per-box error {e:.2e}")
    assert e < FP32_BOX, e


@pytest.mark.parametrize("nrhs", [9, 40])
@pytest.mark.parametrize("prec", [1, 2])
def test_blr_many_boxes(prec, nrhs):
    """128 boxes, whose projections and expansions are both launched with one
    wave per item (from 1024 items on), one and several column groups, the last
    one partial."""
    need_gpu()
    n, parts, ov, pmax, eps = (48, 48, 8), (8, 8, 2), 2, 4, 1e-3
    w = wl.small_random(n, npml=2, q=60.0, seed=9, parts=parts, overlap=ov)
    say(f"blr many boxes prec={prec} nrhs={nrhs}")
    M = oblr.OrasBLR(oracle_fields(w), parts, ov, eps, pmax)
    for k in range(M.subs[0].hi[2] - M.subs[0].lo[2]):
        proj, exp = np.zeros(8), np.zeros(8)      # items of the boxes that share a die
        for j, sol in enumerate(M.solvers):
            r = sol.inv[k].rank
            low = np.where((r >= 0) & ~np.eye(len(r), dtype=bool), r, 0).sum(axis=0)
            proj[j % 8] += -(-low // 32).sum()
            exp[j % 8] += len(r)
        assert 8 * proj.max() >= 1024 and 8 * exp.max() >= 1024
    S = setup(w, prec=prec, parts=parts, overlap=ov)
    assert S.compress(eps, pmax)["lowrank"] > 0
    x = rand_field((w.nz, w.ny, w.nx), nrhs, 17)
    e = box_err(S.apply_M(to_dev(x, S)).cpu().numpy(), M.apply(x), parts, ov)
    say(f"  per-box error {e:.2e}")
    assert e < (BLR32_BOX * eps if prec == 1 else FP64_BOX), e
