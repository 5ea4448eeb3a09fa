"""Direct product on both sides of the lines where a lane takes one, two or four
receivers (20,000 sources: 1665 and 3329 receivers), with whole and ragged groups
of receivers.

Bound: FP64 sums of 20,000 terms against the oracle's, 1e-12 of the largest value
(the bound of test_gpu_direct.py)."""
import numpy as np
import pytest

import oracle
from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr", [1664, 1665, 1791, 3328, 3329, 3583, 3585])
def test_receivers_per_lane(nr):
    import torch
    n = 20000
    cl = wl.cluster(32, 3, 30.0, 0.5, 1.0, 0.5, 17, perturb=0.05)
    s, nrm, _ = oracle.geometry(cl.xyz, cl.tri)
    rng = np.random.default_rng(nr)
    xyz, s, nrm = cl.xyz[:n], s[:n], nrm[:n]
    x, y = rng.uniform(-1, 1, (2, n))
    rows = rng.integers(0, n, nr)
    dev = [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in (xyz, s, nrm, x, y, rows)]
    for f, g in ((1.0, 0.0), (0.0, 1.0), (0.7, -1.3)):
        ref = oracle.offdiag_mvp(xyz, s, nrm, f, x if f else None, g, y if g else None, rows=rows)
        out = bfm.direct_dev(dev[0], dev[1], dev[2], f, dev[3] if f else None, g, dev[4] if g else None, dev[5])
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref)), (f, g)
