"""Work items of the symmetric near field: a shape that the caller asks for is
the one that runs, whatever the mesh's size; the rule by size stands in for -1
alone."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

SHAPES = [(256, 128, 192), (128, 128, 128), (256, 128, 384)]


@pytest.mark.parametrize("points", [1, 642, 524287, 524288, 3210000])
def test_the_option_decides(points):
    assert [bfm.debug_near_shape(points, k) for k in range(3)] == SHAPES
    assert bfm.debug_near_shape(points, -1) == ((128, 64, 64) if points < 524288 else SHAPES[0])


def test_other_shapes_are_refused():
    for shape in (-2, 3):
        with pytest.raises(bfm.BfmError) as e:
            bfm.debug_near_shape(642, shape)
        assert e.value.code == -1


@pytest.mark.gpu
@pytest.mark.parametrize("lmax,low,high", [(4, 65, 128), (3, 257, 512), (2, 513, 768)])
@pytest.mark.parametrize("prec", [bfm.PREC_FP64, bfm.PREC_FP32])
def test_shapes_agree_on_large_leaves(lmax, low, high, prec):
    """Leaves of up to 127, 496 and 645 points, so that a lane holds one
    to four receivers and an item's sources run over several tiles. The shapes
    regroup the same pair sums: FP64 products agree to rounding (1e-12 of the
    largest value), FP32 ones to FP32 rounding of sums of a few thousand terms of
    one sign (2e-6)."""
    cl = wl.cluster(7, 3, 12.0, 0.5, 1.0, 0.5, seed=19, perturb=0.05)
    x = 1.0 + 0.5 * np.cos(np.arange(cl.nv) * 0.37)
    ys = []
    for shape in (1, 0, 2, -1):
        sv = bfm.Solver(p=12, p_lo=12, lmax=lmax, p2p_shape=shape)
        sv.set_cluster(cl)
        assert low <= sv.tree_stats()["max_leaf"] <= high, sv.tree_stats()
        ys.append(sv.matvec(1.0, x, precision=prec))
        sv.close()
    for y in ys[1:]:
        assert np.max(np.abs(y - ys[0])) / np.max(np.abs(ys[0])) < (1e-12 if prec == bfm.PREC_FP64 else 2e-6)


@pytest.mark.gpu
def test_autotuned_shape_is_one_that_was_timed():
    """On a small mesh the rule by size and the three shapes are different items,
    each a candidate; the choice is stored and survives a second call."""
    cl = wl.cluster(3, 2, 10.0, 0.5, 1.0, 0.5, seed=4, perturb=0.05)
    n = {}
    for shape in (-1, 1):
        sv = bfm.Solver(p2p_shape=shape)
        sv.set_cluster(cl)
        r = sv.autotune(1e-6)
        n[shape] = r["candidates"]
        assert -1 <= r["p2p_shape"] <= 2 and sv.opt.p2p_shape == r["p2p_shape"]
        if shape == 1:
            assert r["p2p_shape"] == 1
        sv.close()
    assert n[-1] == n[1] + 4
