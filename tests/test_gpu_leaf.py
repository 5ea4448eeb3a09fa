"""P2M and L2P at the leaf sizes and item counts where their split changes
(one to four points a lane, several items per leaf, orders or points split
over the waves), against the all-pairs sum on the GPU.

Bounds: those of test_gpu_parity.py's fixed-depth products (truncation where
nearly every far interaction is at the minimum separation, 3e-6 and 2e-5 for
the single and the double layer in the 2-norm, 1.5e-5 and 1e-4 of the largest
value); a lost or doubled point or order shows as an error of order one. FP32:
3e-5 (test_gpu_mixed.py)."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,level,lmax", [(1, 3, 2), (2, 4, 2), (6, 4, 2), (40, 3, 3), (400, 2, 5), (700, 2, 6)])
def test_products_match_direct(nb, level, lmax):
    cl = wl.cluster(nb, level, 9.0 * max(nb, 2) ** (1 / 3), 0.5, 1.0, 0.5, 50 + nb, perturb=0.05)
    rng = np.random.default_rng(nb)
    x, y = rng.uniform(-1, 1, cl.nv), rng.uniform(-1, 1, cl.nv)
    sv = bfm.Solver(p=20, p_diag=20, lmax=lmax)
    sv.set_cluster(cl)
    st = sv.tree_stats()
    for f, g, tol, most in ((1.0, 0.0, 3e-6, 1.5e-5), (0.0, 1.0, 2e-5, 1e-4), (0.5, 2.0, 2e-5, 1e-4)):
        a = sv.matvec(f, x if f else None, g, y if g else None)
        b = sv.matvec(f, x if f else None, g, y if g else None, direct=True)
        err, largest = np.linalg.norm(a - b) / np.linalg.norm(b), np.max(np.abs(a - b)) / np.max(np.abs(b))
        print(f"nb={nb} lmax={lmax} leaves={st['leaves']} max_leaf={st['max_leaf']} f={f} g={g}: {err:.2e} {largest:.2e}")
        assert err < tol and largest < most
    # low precision at the same sizes
    a = sv.matvec(1.0, x, precision=bfm.PREC_FP32)
    b = sv.matvec(1.0, x, direct=True)
    assert np.linalg.norm(a - b) < 3e-5 * np.linalg.norm(b)
    sv.close()
