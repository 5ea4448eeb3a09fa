"""Meshes on which the first steps of a cycle orthogonalise in one workgroup and the
later ones in four launches (up to 32, 19, 12 and 3 vectors in one), against a
restart length that stays with one kind of step.

Bound of test_gpu_gmres.py: every run stops at a true relative residual of 1e-12
and the condition number is below 100, so two runs agree to 2e-10."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,level", [(6, 2), (2, 3), (10, 2), (25, 2)])
def test_steps_of_both_kinds_in_a_cycle(nb, level):
    cl = wl.cluster(nb, level, 9.0 * max(nb, 2) ** (1 / 3), 0.5, 1.0, 0.5, 7 + nb, perturb=0.05)
    phi = wl.rough_phi(cl, 3)
    q = {}
    for restart in (2, 13, 20, 40):
        sv = bfm.Solver(p=8, p_diag=8, leaf_target=32, gmres_tol=1e-12, gmres_restart=restart, gmres_maxit=6000)
        sv.set_cluster(cl)
        q[restart], info = sv.solve(phi)
        sv.close()
        assert info["converged"] and info["rel_residual"] <= 1e-12
        err = np.linalg.norm(q[restart] - q[2]) / np.linalg.norm(q[2])
        assert err < 2e-10, (restart, err, info)
