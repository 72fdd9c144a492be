"""Aggregation of rows at any alignment: offsets of one element, odd strides
and widths around the 4-feature lanes, for every input type, against the oracle
(the bound of test_gpu_parity: 1e-5 of the sum of |terms|)."""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_close, bf16_bits, bf16_round, dev, host, note

pytestmark = pytest.mark.gpu

N = 3000


@pytest.fixture(scope="module")
def graph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2411_16025_amd as G
    G.lib()
    src, dst = synth.rmat_edges(61, N, 40000, perm_seed=62)
    flags = G.GCN_SYMMETRIZE | G.GCN_ADD_SELF_LOOPS
    g = G.gcn_build_csr(N, N, dev(src), dev(dst), flags)
    G.gcn_normalize(g)
    return G, g, oracle.Graph(N, N, src, dst, flags, deg=None, normalized=True)


def _shifted(torch, a, off, ld):
    """The matrix a at element offset off of a buffer with rows ld apart."""
    buf = torch.zeros(off + N * ld, dtype=a.dtype, device="cuda:0")
    v = buf[off:].view(N, ld)[:, :a.shape[1]]
    v.copy_(a)
    return v


@pytest.mark.parametrize("F", [1, 3, 4, 5, 6, 7, 17, 61, 127, 129, 131])
def test_rows_at_any_offset(graph, F):
    import torch
    G, g, og = graph
    x = synth.normal(63, N, F)
    xb = bf16_round(x)
    for off, pad in ((0, 0), (1, 0), (3, 1), (1, 2)):
        note("unaligned F=%d offset %d pad %d" % (F, off, pad))
        Y = torch.full((N, F + pad + 1), 7.0, device="cuda:0")
        G.gcn_aggregate_fwd(g, _shifted(torch, dev(x), off, F + pad), Y=Y[:, :F])
        ref, S = og.fwd(x)
        y = host(Y)
        assert_close(y[:, :F], ref, S, what="f32")
        assert np.all(y[:, F:] == 7.0)
        b = torch.from_numpy(bf16_bits(x).view(np.int16)).view(torch.bfloat16).to("cuda:0")
        ref, S = og.bwd(xb)
        assert_close(host(G.gcn_aggregate_bwd(g, _shifted(torch, b, off, F + pad))), ref, S,
                     what="bf16")


@pytest.mark.parametrize("bits", [8, 2])
@pytest.mark.parametrize("F", [3, 4, 5, 6, 7, 61, 130])
def test_codes_at_any_offset(graph, F, bits):
    import torch
    G, g, og = graph
    n_loc = N - 800
    x = synth.normal(64, N, F)
    q, zmin, scale = G.gcn_layernorm_quantize(dev(x[n_loc:]), bits=bits, layernorm=False)
    codes = host(q)
    if bits == 2:
        codes = np.stack([(codes >> s) & 3 for s in (0, 2, 4, 6)], 2).reshape(len(codes), -1)[:, :F]
    full = x.astype(np.float64)
    full[n_loc:] = codes * host(scale)[:, None].astype(np.float64) + host(zmin)[:, None]
    ref, S = og.fwd(full.astype(np.float32))
    for off, pad in ((0, 0), (1, 0), (3, 1)):
        note("unaligned codes F=%d bits=%d offset %d pad %d" % (F, bits, off, pad))
        ldq = q.shape[1] + pad
        buf = torch.zeros(off + 800 * ldq, dtype=torch.uint8, device="cuda:0")
        qs = buf[off:].view(800, ldq)[:, :q.shape[1]]
        qs.copy_(q)
        X = torch.zeros(1 + n_loc * (F + 1), device="cuda:0")[1:].view(n_loc, F + 1)[:, :F]
        X.copy_(dev(x[:n_loc]))
        Y = G.gcn_aggregate_fwd_q8halo(g, n_loc, X, qs, zmin, scale, F=F, bits=bits)
        # rounding the dequantized rows to fp32 for the oracle is within 2^-24 of each term
        assert_close(host(Y), ref, S, what="codes")
