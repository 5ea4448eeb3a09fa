"""Preconditioned solves where the preconditioner's tiles and runs end: template
meshes smaller than a run of loads (12 vertices), degrees with fewer coefficients
than one, 16 x 16 and 48 x 16 coefficient tiles, 16 and 32 bubbles a wave, against
the same systems solved without a preconditioner.

Tolerance: both solutions have a relative residual below 1e-10; the single-layer
systems of these small clusters of unit-scale spheres have condition numbers of
a few hundred at most, so they agree to 1e-7 of the largest value."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,level,degree", [(1, 0, 1), (3, 0, 2), (17, 1, 2), (5, 2, 3), (33, 1, 4), (511, 0, 2),
                                             (513, 1, 4), (2047, 0, 2), (2049, 0, 2), (2050, 1, 3)])
def test_preconditioned_solution_is_the_same(nb, level, degree):
    cl = wl.cluster(nb, level, 3.2 * max(2.0, nb ** (1.0 / 3.0)), 0.5, 1.0, 0.5, seed=nb, perturb=0.05)
    phi = wl.smooth_phi(cl, nb + 1)
    q = []
    for pc in (bfm.PRECOND_NONE, bfm.PRECOND_SH_COARSE):
        sv = bfm.Solver(p=8, gmres_tol=1e-10, gmres_maxit=2000, precond=pc, precond_degree=degree)
        sv.set_cluster(cl)
        x, info = sv.solve(phi)
        assert info["converged"]
        q.append(x)
    np.testing.assert_allclose(q[1], q[0], rtol=0, atol=1e-7 * np.abs(q[0]).max())
