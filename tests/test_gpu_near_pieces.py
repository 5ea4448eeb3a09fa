"""One-sided near field (both layers, the five-channel diagonal pass) at source
lists just below, at and just above its pieces of 128 sources: a convex mesh of n
vertices inside one leaf, whose list is then the mesh itself, and a tetrahedron
in the opposite corner of the cube. Up to 128 sources every sum is stored by one
work item, above them several add theirs; 130 sources are two pieces of 65, 257
three of 86, neither a multiple of the 64-source tile.

Tolerance: against all pairs in FP64. The two leaves lie 5.2 box sides apart, so
at order 20 the far field is exact to (0.87 / 4.33)^20 = 1e-14 of it, and the sums
are of at most 257 terms whose magnitudes add up to less than 1e3 times the largest
result: 257 eps 1e3 = 6e-11, taken as 1e-10 of the largest value."""
import numpy as np
import pytest
from scipy.spatial import ConvexHull

import oracle
from paper_1905_01341_amd import bfm

pytestmark = pytest.mark.gpu


def convex(n, seed):
    """n points spread over a sphere and the outward triangles of their hull."""
    k = np.arange(n) + 0.5
    z, a = 1.0 - 2.0 * k / n, k * np.pi * (1.0 + 5.0 ** 0.5)
    r = np.sqrt(1.0 - z * z)
    v = np.stack([r * np.cos(a), r * np.sin(a), z], 1) + 0.01 * np.random.default_rng(seed).standard_normal((n, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    tri = ConvexHull(v).simplices.copy()
    c = np.cross(v[tri[:, 1]] - v[tri[:, 0]], v[tri[:, 2]] - v[tri[:, 0]])
    flip = (c * v[tri].sum(1)).sum(1) < 0
    tri[flip] = tri[flip][:, [0, 2, 1]]
    assert len(tri) == 2 * n - 4
    return v, tri


@pytest.mark.parametrize("n", [64, 65, 127, 128, 129, 130, 255, 256, 257])
def test_around_the_pieces(n):
    v, tri = convex(n, n)
    t, ttri = convex(4, 1)
    xyz = np.concatenate([0.4 * v + 0.5, 0.4 * t + 7.5])
    tri = np.concatenate([tri, ttri + n]).astype(np.int32)
    sv = bfm.Solver(p=20, p_diag=20, lmax=2)
    sv.set_mesh(xyz, tri, np.array([0, n, n + 4], np.int64), np.array([0, 2 * n - 4, 2 * n], np.int64))
    st = sv.tree_stats()
    assert st["leaves"] == 2 and st["max_leaf"] == n and st["near_pairs"] == n * n + 16, st
    rng = np.random.default_rng(n)
    x, y, phi = rng.standard_normal((3, n + 4))
    for f, g in ((1.0, 0.7), (0.0, -1.3)):
        a, b = sv.matvec(f, x, g, y), sv.matvec(f, x, g, y, direct=True)
        np.testing.assert_allclose(a, b, rtol=0, atol=1e-10 * np.abs(b).max())
    m, l, b = sv.diagonals(phi)
    s, nrm, _ = oracle.geometry(xyz, tri)
    d = oracle.sums(xyz, s, nrm, phi)
    mr, lr, _ = oracle.diagonals(xyz, s, nrm, sm=d)
    br = oracle.rhs(phi, d["B"])
    assert np.abs(m - mr).max() < 1e-10 * 0.5
    np.testing.assert_allclose(l, lr, rtol=0, atol=1e-10 * np.abs(lr).max())
    np.testing.assert_allclose(b, br, rtol=0, atol=1e-10 * np.abs(br).max())
