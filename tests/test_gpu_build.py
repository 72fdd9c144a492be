"""Graph construction at the edges of its tiles (4096 keys, 1024 per wavefront),
with duplicates across them, few distinct digits, and rows mostly empty (the row
search of the normalization): bit-exact against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, note

pytestmark = pytest.mark.gpu

LOOPS, SYM = 2, 1


def _check(n_rows, n_cols, src, dst, flags, deg=None):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2411_16025_amd as G
    g = G.gcn_build_csr(n_rows, n_cols, dev(src), dev(dst), flags)
    G.gcn_normalize(g, dev(deg) if deg is not None else None)
    og = oracle.Graph(n_rows, n_cols, src, dst, flags, deg=deg)
    for which, (p, i, v) in ((0, (og.csr_ptr, og.csr_idx, og.csr_val)),
                             (1, (og.csc_ptr, og.csc_idx, og.csc_val))):
        ptr, idx, val = G.gcn_graph_export(g, which)
        assert np.array_equal(ptr, p)
        assert np.array_equal(idx, i)
        assert np.array_equal(val.view(np.int32), v.view(np.int32))


@pytest.mark.parametrize("m", [0, 1, 63, 64, 65, 1023, 1025, 4095, 4096, 4097, 8191, 8193, 50001])
def test_key_counts(m):
    note("build: %d keys" % m)
    n = 700
    src, dst = synth.er_edges(81, n, m) if m else (np.zeros(0, np.int32), np.zeros(0, np.int32))
    _check(n, n, src, dst, 0)
    _check(n, n, src, dst, SYM | LOOPS)


@pytest.mark.parametrize("n,copies", [(3, 3000), (40, 997), (5000, 3)])
def test_duplicates_across_tiles(n, copies):
    note("build: duplicates n=%d x %d" % (n, copies))
    src, dst = synth.er_edges(82, n, 2 * n)
    src, dst = np.tile(src, copies), np.tile(dst, copies)
    p = synth.permutation(83, len(src))
    _check(n, n, src[p], dst[p], LOOPS)


@pytest.mark.parametrize("rows", [2047, 2048, 2049, 300000])
def test_rows_mostly_empty(rows):
    """A tile of the normalization spans few, 2,048 and many more rows."""
    note("build: %d mostly empty rows" % rows)
    rng = np.random.default_rng(84)
    m = 2500
    src = rng.integers(0, 50000, m).astype(np.int32)
    dst = np.sort(rng.choice(rows, size=m)).astype(np.int32)
    dst[0], dst[-1] = 0, rows - 1
    deg = rng.integers(0, 2 ** 31 - 1, max(rows, 50000)).astype(np.int32)
    _check(rows, 50000, src, dst, 0, deg=deg)
