"""The gradient kernel at the edges of its 16 x 4 x 4 node tiles and its
right-hand-side loop, against the oracle's gradient of the same fields."""
import numpy as np
import pytest

from oracle import adjoint
from paper_2110_15113_amd import workloads as wl

from gpu_util import need_gpu, oracle_fields, rand_field, say, setup, to_dev

pytestmark = pytest.mark.gpu


# one node more and less than whole tiles, a tile partly outside, one tile
@pytest.mark.parametrize("n", [(16, 8, 4), (17, 5, 9), (15, 7, 3), (33, 3, 5), (3, 4, 13)])
@pytest.mark.parametrize("nrhs", [1, 2, 5])
def test_gradient_tiles(n, nrhs):
    need_gpu()
    say(f"gradient {n} nrhs={nrhs}")
    w = wl.small_random(n, npml=1, q=60.0, seed=41)
    F = oracle_fields(w)
    u, mu = rand_field(F.shape, nrhs, 42), rand_field(F.shape, nrhs, 43)
    S = setup(w)
    for weights, ref in ((False, adjoint.gradient(F, u, mu)),
                         (True, adjoint.gradient_exact(F, u, mu, 1.0 / w.vel ** 2))):
        g = S.gradient(to_dev(u, S), to_dev(mu, S), weights=weights).cpu().numpy()
        # the bar of the gradient's other comparisons with the oracle
        assert np.abs(g - ref).max() < 1e-11 * np.abs(ref).max()


# tiles of 4 x 8 x 8 nodes up to 8 nodes along x, at their edges
@pytest.mark.parametrize("n", [(4, 8, 8), (5, 9, 7), (8, 17, 9), (9, 8, 8)])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_gradient_tiles_of_narrow_grids(n, nrhs):
    test_gradient_tiles(n, nrhs)


def test_gradient_of_more_tiles_than_a_launch_holds():
    """Half a billion nodes, few of them along two axes, whose tiles may need
    2^32 threads.  The fields repeat along z, so away from the ends the gradient
    repeats that of a short grid, tile by tile."""
    need_gpu()
    import torch
    if torch.cuda.mem_get_info()[0] < 150e9:
        pytest.skip("needs 150 GB of device memory")
    from paper_2110_15113_amd import oras
    period, ny, nx = 64, 5, 3
    rng = np.random.default_rng(44)
    fields = [rng.normal(size=(1, period, ny, nx)) + 1j * rng.normal(size=(1, period, ny, nx))
              for _ in range(2)]
    inner = []
    for nz in (3 * period, 524300 * period):
        say(f"gradient of {nx} x {ny} x {nz} nodes")
        S = oras.Solver(0)
        S.assemble(torch.full((nz, ny, nx), 2000.0, dtype=torch.float64, device=S.device), 20.0, 0, 40.0)
        u, mu = (to_dev(f, S).repeat(1, nz // period, 1, 1) for f in fields)
        g = S.gradient(u, mu, weights=True)
        inner.append(g[period:-period].view(-1, period, ny, nx))
        S.close()
    assert bool((inner[0] != 0).all())
    assert bool((inner[1] == inner[0]).all())
