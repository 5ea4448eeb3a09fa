"""The Arnoldi orthogonalisation's paths (one workgroup, fused passes, more
vectors than a fused pass holds) at the sizes where they change.

A solve's answer does not depend on the restart length: every run stops at a
true relative residual of 1e-12, so two runs differ by at most the two
residuals times the system's condition number (below 100 for these
clusters): 2e-10."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,level", [(1, 1), (2, 2), (6, 3), (7, 3), (30, 3)])
def test_restart_lengths_agree(nb, level):
    cl = wl.cluster(nb, level, 9.0 * max(nb, 2) ** (1 / 3), 0.5, 1.0, 0.5, 7 + nb, perturb=0.05)
    phi = wl.rough_phi(cl, 3)
    ref = None
    for restart in (30, 4, 8, 9, 16, 17, 32, 33, 128):
        sv = bfm.Solver(p=8, p_diag=8, leaf_target=32, gmres_tol=1e-12, gmres_restart=restart, gmres_maxit=4000)
        sv.set_cluster(cl)
        q, info = sv.solve(phi)
        q2, info2 = sv.solve(phi, q0=q)  # from the solution: no iteration needed
        q0, info0 = sv.solve(np.zeros(cl.nv), q0=q)  # b = 0: the zero solution
        sv.close()
        assert info["converged"] and info["rel_residual"] <= 1e-12
        assert info2["iterations"] == 0 and info2["matvecs"] == 1 and np.array_equal(q2, q)
        assert info0["converged"] and not np.any(q0)
        if ref is None:
            ref = q
        err = np.linalg.norm(q - ref) / np.linalg.norm(ref)
        assert err < 2e-10, (restart, err, info)
