"""Near field of the product with both layers, against the sum of the two
single-layer products: its monopole part against the symmetric pair kernel, at
leaf occupancies around its 64- and 128-receiver chunks, 64-source tiles and
384-source pieces.

Tolerance: the product is linear, so the two sides differ by rounding alone: sums
of at most a few thousand terms of either sign, about sqrt(3000) eps = 1.2e-14
of the sum of magnitudes, which for random densities exceeds the result by at
most a factor of 100 here: 1e-12 of the largest value."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,level,leaf", [(1, 0, 64), (1, 1, 64), (1, 3, 8), (3, 2, 64), (7, 2, 128), (5, 3, 400),
                                           (2, 3, 1000)])
def test_both_layers_are_the_sum_of_each(nb, level, leaf):
    cl = wl.cluster(nb, level, 3.0 * max(2.0, nb ** (1.0 / 3.0)), 0.5, 1.0, 0.5, seed=nb + level, perturb=0.05)
    sv = bfm.Solver(p=12, leaf_target=leaf)
    sv.set_cluster(cl)
    rng = np.random.default_rng(leaf)
    x, y = rng.standard_normal((2, sv.nv))
    both = sv.matvec(1.0, x, 0.7, y)
    each = sv.matvec(1.0, x) + sv.matvec(0.0, None, 0.7, y)
    np.testing.assert_allclose(both, each, rtol=0, atol=1e-12 * np.abs(each).max())
