"""FP64 M2L with the azimuth rotated out (csrc/fmm_azim.hip) against the
rotation-factored M2L, an independent kernel with its own operators (checked
against the oracle in test_gpu_rot.py), for every launch shape and order at
sizes with empty, partial and single-column tiles.

Tolerance: both forms are exact factorings of one operator, so their products
differ by the rounding of sums of at most a few thousand terms of the result's
size: 1e-12 of the largest value, the bound of test_gpu_rot.py."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


def maxrel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("nb,level,leaf", [(1, 2, 8), (5, 3, 40)])
@pytest.mark.parametrize("p", [4, 8, 12, 16, 20])
@pytest.mark.parametrize("shape", [-1, 0, 1, 2])
def test_shapes_match_rotation_factored(nb, level, leaf, p, shape):
    cl = wl.cluster(nb, level, 8.0, 0.5, 1.0, 0.5, 31 + nb, perturb=0.05)
    x, y = np.cos(np.arange(cl.nv) * 0.37), np.sin(np.arange(cl.nv) * 0.71)
    res = []
    for sh in (shape, 3):
        sv = bfm.Solver(p=p, p_diag=p, leaf_target=leaf, m2l_shape=sh, m2l_orders=1)
        sv.set_cluster(cl)
        first = sv.matvec(1.0, x, 1.0, y)
        res.append((first, sv.matvec(1.0, x, 1.0, y), *sv.diagonals(x)))
        assert sv.tree_stats()["m2l_pairs"] > 0
        sv.close()
    (a, a2, *da), (b, _, *db) = res
    print(f"nb={nb} p={p} shape={shape}: {maxrel(a, b):.2e}")
    assert maxrel(a, b) < 1e-12 and maxrel(a2, a) < 1e-12
    # M_ii against the 1/2 it is a difference from, L_ii and b by their largest
    assert np.abs(da[0] - db[0]).max() / 0.5 < 1e-12
    assert maxrel(da[2], db[2]) < 1e-12 and maxrel(da[1], db[1]) < 1e-11
