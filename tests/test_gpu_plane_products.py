"""Every split of the plane products (column blocks, rows and waves per
work-group) against the oracle's local solves, box by box."""
import functools

import pytest

from oracle import oras as ooras
from paper_2110_15113_amd import workloads as wl

from gpu_util import (FP32_BOX, FP64_BOX, box_err, need_gpu, oracle_fields, rand_field, say, setup,
                      to_dev)

pytestmark = pytest.mark.gpu

# few subdomains; 288 of them, whose products take the splits of large launches
GRIDS = {"few": dict(n=(17, 15, 14), parts=(2, 2, 1), ov=2),
         "many": dict(n=(36, 36, 24), parts=(6, 6, 8), ov=2)}
PADDED = 56


@functools.lru_cache(maxsize=None)
def reference(grid, columns=PADDED):
    c = GRIDS[grid]
    w = wl.small_random(c["n"], npml=2, q=70.0, seed=31)
    x = rand_field((w.nz, w.ny, w.nx), columns, 33)
    return w, x, ooras.ORAS(oracle_fields(w), c["parts"], c["ov"]).apply(x)


# padded to 8, 16, 24, 32, 40, 48 and 56 columns
@pytest.mark.parametrize("nrhs", [1, 16, 19, 32, 35, 47, 56])
@pytest.mark.parametrize("grid", list(GRIDS))
def test_plane_products_c128(grid, nrhs):
    need_gpu()
    say(f"plane products c128 {grid} nrhs={nrhs}")
    c = GRIDS[grid]
    w, x, ref = reference(grid)
    S = setup(w, prec=2, parts=c["parts"], overlap=c["ov"])
    y = S.apply_M(to_dev(x[:nrhs], S)).cpu().numpy()
    assert box_err(y, ref[:nrhs], c["parts"], c["ov"]) < FP64_BOX


# one, two chunks of 32 columns, the last one partial
@pytest.mark.parametrize("nrhs", [1, 32, 47])
@pytest.mark.parametrize("grid", list(GRIDS))
def test_plane_products_c64(grid, nrhs):
    need_gpu()
    say(f"plane products c64 {grid} nrhs={nrhs}")
    c = GRIDS[grid]
    w, x, ref = reference(grid)
    S = setup(w, prec=1, parts=c["parts"], overlap=c["ov"])
    y = S.apply_M(to_dev(x[:nrhs], S)).cpu().numpy()
    assert box_err(y, ref[:nrhs], c["parts"], c["ov"]) < FP32_BOX


# planes of one row tile in 2048 boxes, of eight in 128, of eleven in one box
# whose 256 columns of t are 1 MB: one and two waves, both row splits
GRIDS.update(short=dict(n=(64, 64, 16), parts=(16, 16, 8), ov=0),
             tiles=dict(n=(60, 60, 16), parts=(4, 4, 8), ov=0),
             one=dict(n=(19, 18, 6), parts=(1, 1, 1), ov=0))


@pytest.mark.parametrize("prec,bar", [(1, FP32_BOX), (2, FP64_BOX)])
@pytest.mark.parametrize("grid,nrhs", [("short", 3), ("short", 16), ("short", 24), ("short", 128),
                                       ("tiles", 64), ("tiles", 128), ("one", 256)])
def test_plane_products_by_plane_size(grid, nrhs, prec, bar):
    need_gpu()
    say(f"plane products {grid} nrhs={nrhs} prec={prec}")
    c = GRIDS[grid]
    w, x, ref = reference(grid, 256 if grid == "one" else 128)
    S = setup(w, prec=prec, parts=c["parts"], overlap=c["ov"])
    y = S.apply_M(to_dev(x[:nrhs], S)).cpu().numpy()
    e = box_err(y, ref[:nrhs], c["parts"], c["ov"])
    say(f"  per-box error {e:.2e}")
    assert e < bar
