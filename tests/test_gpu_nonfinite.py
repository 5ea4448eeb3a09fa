"""A solve whose residual is not a number does not report convergence: the
iteration limit ends it, the flag stays off and the residual comes back as it is."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,level", [(1, 1), (7, 3)])  # one-workgroup and fused Arnoldi steps
@pytest.mark.parametrize("form", [dict(), dict(precision=bfm.PREC_BF16X3, p_lo=8),
                                  dict(precond=bfm.PRECOND_SH_COARSE, precond_degree=2)])
def test_guess_that_is_not_a_number(nb, level, form):
    cl = wl.cluster(nb, level, 18.0, 0.5, 1.0, 0.5, 5 + nb, perturb=0.05)
    phi = wl.smooth_phi(cl, 6)
    sv = bfm.Solver(p=8, gmres_tol=1e-8, gmres_maxit=3, **form)
    sv.set_cluster(cl)
    q0 = np.ones(cl.nv)
    q0[cl.nv // 2] = np.nan
    q, info = sv.solve(phi, q0=q0, check=False)
    assert not info["converged"] and np.isnan(info["rel_residual"]) and info["iterations"] == 3
    with pytest.raises(bfm.BfmError) as e:
        sv.solve(phi, q0=q0)
    assert e.value.code == -4
    # the handle is as good as new
    sv.set_options(gmres_maxit=300)
    q, info = sv.solve(phi)
    assert info["converged"] and np.all(np.isfinite(q))
