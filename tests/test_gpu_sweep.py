"""GPU inverse of a symmetric positive definite matrix (the coarse correction
of the two-level preconditioner) at the edges of its blocked sweep: pivot
blocks of 128, update tiles of 64, panels of 32 rows.

Tolerance: eigenvalues of the test matrices lie in [1, 5], so every Schur
complement of the sweep is at least 1 and each of the n pivots changes an
element by a rounding error of at most about 25 eps; n eps 25 is 2e-12 at the
largest n here. The result is symmetric to the bit (one triangle is computed
and mirrored)."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 31, 63, 65, 127, 128, 129, 160, 191, 192, 193, 255, 256, 257, 320, 385])
def test_inverse_at_block_edges(n):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, n))
    A = X @ X.T / n + np.eye(n)
    Ai = bfm.debug_spd_inverse(A)
    ref = np.linalg.inv(A)
    np.testing.assert_allclose(Ai, ref, rtol=0, atol=2e-12)
    np.testing.assert_array_equal(Ai, Ai.T)
