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
