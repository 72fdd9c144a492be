"""One launch for all rows: every route of small and mid-size matrices on both
sides of its limits (rows and feature tiles in flight, rows of 64, 256 and 2,048
entries, slots of at most 8 lanes, gathered features), against the oracle within
1e-5 of the sum of |terms|, and the same bits on a second run."""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_close, dev, host, note

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 3, 16, 17, 32, 33, 63, 64, 65, 128, 255, 256, 257, 2047, 2048, 2049, 4097]


def _graph(n, long_rows):
    """Rows of the lengths above (without long_rows: up to 64), several of
    each, among random short ones."""
    rng = np.random.default_rng(71)
    src, dst = synth.er_edges(72, n, 3 * n)
    keep = dst >= 200
    src, dst = [src[keep]], [dst[keep]]
    lens = [k for k in LENGTHS if k <= n and (long_rows or k <= 64)]
    for r in range(min(200, n)):
        k = lens[r % len(lens)]
        src.append(rng.choice(n, size=k, replace=False).astype(np.int32))
        dst.append(np.full(k, r, np.int32))
    return np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)


# (rows, long rows, widths): 4,096 / 4,097 rows without long rows; as many rows
# and tiles with them: one, two (F > 128) and three tiles; a large one on a launch per class
CASES = [(1, True, [1, 64]), (300, True, [3, 16, 32, 36, 64]), (4096, False, [16, 64, 128, 132]),
         (4097, False, [64]), (5461, True, [300]), (2048, True, [128, 132]), (2049, True, [132]),
         (16384, True, [16, 47, 128]), (16385, True, [4, 16, 32, 36, 128]), (90000, True, [16, 100])]


@pytest.mark.parametrize("n,long_rows,widths", CASES)
def test_rows_routes(n, long_rows, widths):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2411_16025_amd as G
    src, dst = _graph(n, long_rows)
    og = oracle.Graph(n, n, src, dst, 0, normalized=False)
    g = G.gcn_build_csr(n, n, dev(src), dev(dst), 0)
    for F in widths:
        note("rows routes n=%d F=%d" % (n, F))
        x = synth.normal(73, n, F)
        for fn, ref in ((G.gcn_aggregate_fwd, og.fwd), (G.gcn_aggregate_bwd, og.bwd)):
            y = fn(g, dev(x))
            r, S = ref(x)
            assert_close(host(y), r, S, what=fn.__name__)
            assert torch.equal(y.view(torch.int32), fn(g, dev(x)).view(torch.int32))


def test_many_gathers():
    """More than 8e8 gathered features: a launch per class, without column blocks."""
    import torch
    import paper_2411_16025_amd as G
    note("rows routes, a launch per class")
    n, F = 200000, 128
    src, dst = synth.rmat_edges(74, n, 3600000, perm_seed=75)
    g = G.gcn_build_csr(n, n, dev(src), dev(dst), G.GCN_SYMMETRIZE)
    assert g.nnz * F > 800000000
    x = synth.normal(76, n, F)
    og = oracle.Graph(n, n, src, dst, G.GCN_SYMMETRIZE, normalized=False)
    y = G.gcn_aggregate_fwd(g, dev(x))
    r, S = og.fwd(x)
    assert_close(host(y), r, S, what="fwd")
