"""Kernels at the sizes where their tiles, splits and remainders change: the
direct product (receivers per lane, tiles of 256 sources, source splits) and
the network's gradient (row tiles, K splits), against the oracle."""
import numpy as np
import pytest

import oracle
from oracle import learned as ol
from oracle import mlp as om
from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl

pytestmark = pytest.mark.gpu

SIZES = [174, 512, 512, 512, 81]


@pytest.mark.parametrize("n", [1, 63, 255, 257, 642, 3210])
@pytest.mark.parametrize("nr", [1, 64, 65, 128, 129, 256, 257, 700])
def test_direct_sizes(n, nr):
    """Bound: sums of at most 3210 terms whose 1/r has a few roundings, 1e-12
    of the largest value (the bound of test_gpu_direct.py)."""
    import torch
    cl = wl.cluster(5, 3, 8.0, 0.5, 1.0, 0.5, 91, perturb=0.05)
    s, nrm, _ = oracle.geometry(cl.xyz, cl.tri)
    rng = np.random.default_rng(1000 * n + nr)
    at = np.sort(rng.choice(cl.nv, size=n, replace=False))
    xyz, s, nrm = cl.xyz[at], s[at], nrm[at]
    x, y = rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
    rows = rng.integers(0, n, nr)
    dev = [torch.tensor(np.ascontiguousarray(a), device="cuda:0") for a in (xyz, s, nrm, x, y, rows)]
    for f, g in ((1.0, 0.0), (0.0, 1.0), (0.7, -1.3)):
        ref = oracle.offdiag_mvp(xyz, s, nrm, f, x if f else None, g, y if g else None, rows=rows)
        for noalloc in (False, True):
            out = torch.full((nr,), 7.0, dtype=torch.float64, device="cuda:0")
            bfm.direct_dev(dev[0], dev[1], dev[2], f, dev[3] if f else None, g, dev[4] if g else None, dev[5], out,
                           noalloc=noalloc)
            err = np.max(np.abs(out.cpu().numpy() - ref))
            assert err <= 1e-12 * max(np.max(np.abs(ref)), 1e-300), (f, g, noalloc, err)


@pytest.mark.parametrize("rows", [1, 31, 64, 65, 129, 300])
def test_gradient_sizes(rows):
    """Bounds of test_gpu_learned.py's gradient test (BF16 products with FP32
    sums against the oracle that rounds the same operands)."""
    params = om.init(SIZES, seed=5)
    rng = np.random.default_rng(rows)
    params = [(W.astype(np.float32).astype(np.float64), 0.1 * rng.standard_normal(b.shape).astype(np.float32).astype(np.float64))
              for W, b in params]
    x = rng.standard_normal((rows, 174)).astype(np.float32)
    t = rng.standard_normal((rows, 81)).astype(np.float32)
    sv = bfm.Solver()
    sv.mlp_set_params(np.concatenate([np.concatenate([W.ravel(), b]) for W, b in params]).astype(np.float32))
    g, loss = sv.mlp_gradient(x, t)
    sv.close()
    lq = om.loss(params, x, t, rnd=ol.bf16)
    assert abs(loss - lq) <= 1e-3 * lq
    o = 0
    for k, (qw, qb) in enumerate(om.backward(params, x, t, rnd=ol.bf16)):
        for q in (qw, qb):
            a = g[o:o + q.size].reshape(q.shape).astype(np.float64)
            o += q.size
            assert np.linalg.norm(a - q) <= 5e-3 * np.linalg.norm(q), (k, q.shape)
