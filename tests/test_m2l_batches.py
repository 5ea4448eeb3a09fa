"""FP64 M2L lists longer than the workspace of per-task results run in batches:
the batches cover the list once, stay within the workspace, and end where a tile
of columns ends; a long list's products match direct sums; the handle holds no
more than the workspace for them."""
import numpy as np
import pytest

from paper_1905_01341_amd import bfm
from paper_1905_01341_amd import workload as wl


def _tiles(off, nch, width):
    return [-(-int(b - a) * nch // width) for a, b in zip(off[:-1], off[1:])]


@pytest.mark.parametrize("nch", [1, 5])
@pytest.mark.parametrize("width", [16, 64, 128])
def test_batches_cover_the_list(nch, width):
    rng = np.random.default_rng(100 * nch + width)
    for most in (width, width + 1, 3 * width - 1, 3 * width, 1000, 10 ** 9):
        if most < width:
            continue
        for _ in range(40):
            n = rng.integers(0, 6 * width, rng.integers(1, 30)) * rng.integers(0, 2, 1)[0] ** rng.integers(0, 2)
            n = np.where(rng.random(n.size) < 0.3, 0, n)
            off = rng.integers(0, 50) + np.concatenate([[0], np.cumsum(n)])
            lo, op, tile = int(off[0]), 0, 0
            before = np.concatenate([[0], np.cumsum(_tiles(off, nch, width))])
            batches = bfm.debug_m2l_batches(off, nch, width, most)
            for hi, hop, htile in batches:
                assert lo < hi <= lo + most or hi == lo == off[-1]
                # every tile of the batch lies in [lo, hi), and its columns cover it
                g0, g1 = before[op] + tile, before[hop] + htile
                cols = 0
                for g in range(g0, g1):
                    o = int(np.searchsorted(before, g, side="right")) - 1
                    c0 = (g - before[o]) * width
                    c1 = min(c0 + width, int(off[o + 1] - off[o]) * nch)
                    assert off[o] * nch + c0 >= lo * nch and off[o] * nch + c1 <= hi * nch
                    cols += c1 - c0
                assert cols == (hi - lo) * nch
                lo, op, tile = hi, hop, htile
            assert lo == off[-1]


@pytest.mark.gpu
def test_long_list_in_batches():
    """The five-channel pass of 321,000 points at order 20 (1.8 GiB of per-task
    results, 1 GiB of workspace) and an order-20 product, against direct sums at
    sampled rows within the fixed depth's 1e-6; and what the handle takes on the
    device."""
    import oracle
    import torch
    cl = wl.cluster(500, 3, 9.0 * 500 ** (1 / 3), 0.5, 1.0, 0.5, seed=3, perturb=0.05)
    phi = wl.smooth_phi(cl, 4)
    sv = bfm.Solver(p=20, p_diag=20, leaf_target=32)
    sv.set_cluster(cl)
    st = sv.tree_stats()
    results = 8 * 5 * 400 * st["m2l_pairs"]
    free0 = torch.cuda.mem_get_info()[0]
    m, l, b = sv.diagonals(phi)
    q = sv.matvec(1.0, phi)
    held = free0 - torch.cuda.mem_get_info()[0]
    print(f"{st}, per-task results {results / 2**20:.0f} MiB, held {held / 2**20:.0f} MiB")
    assert results > 1.5 * 2 ** 30  # two batches
    # expansions of both groups (multipole and local), the pass's point data, operators
    # and lists, the workspace
    most = 2 * 8 * 400 * 6 * st["boxes"] + 8 * cl.nv * 64 + 2 ** 28 + 2 ** 30
    assert held < most, (held, most)
    s, n, _ = oracle.geometry(cl.xyz, cl.tri)
    rows = np.arange(5, cl.nv, 1201)
    d = oracle.sums(cl.xyz, s, n, phi, rows=rows)
    mr, lr, _ = oracle.diagonals(cl.xyz, s, n, rows=rows, sm=d)
    br = oracle.rhs(phi, d["B"], rows=rows)
    rel = lambda x, y: float(np.linalg.norm(x - y) / np.linalg.norm(y))
    assert np.abs(m[rows] - mr).max() / 0.5 < 1e-6 and rel(l[rows], lr) < 1e-6 and rel(b[rows], br) < 1e-6
    full = sv.matvec(1.0, phi, direct=True)
    assert rel(q, full) < 1e-6
