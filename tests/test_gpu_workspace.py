"""Kept temporaries: calls on several streams and from several threads, and
streams that come and go, give the bits of the same calls one after another."""

import ctypes
import os
import threading

import numpy as np
import pytest

import synth
from gpu_util import dev, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2411_16025_amd as G
    G.lib()
    # a hub of 60,000 entries: chunks and partial rows (temporaries) in every call
    n = 70000
    src = np.concatenate([np.arange(1, 60001), synth.er_edges(1, n, 200000)[0]]).astype(np.int32)
    dst = np.concatenate([np.zeros(60000), synth.er_edges(1, n, 200000)[1]]).astype(np.int32)
    g = G.gcn_build_csr(n, n, dev(src), dev(dst), G.GCN_SYMMETRIZE | G.GCN_ADD_SELF_LOOPS)
    G.gcn_normalize(g)
    X = [dev(synth.normal(40 + k, n, 64)) for k in range(4)]
    W = dev(synth.normal(50, 64, 64))

    def work(k, stream=None):
        y = G.gcn_aggregate_fwd(g, X[k], stream=stream)
        dw = G.gcn_gemm_f32(G.GCN_GEMM_TN, X[k], y, stream=stream)
        return y, G.gcn_gemm_f32(G.GCN_GEMM_NT, y, W, stream=stream), dw

    ref = [work(k) for k in range(4)]
    torch.cuda.synchronize()
    return torch, G, work, ref


def _same(torch, a, b):
    return all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))


def test_streams_and_threads(case):
    torch, G, work, ref = case
    note("workspace: 4 threads, a stream each")
    bad = []

    def run(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(20):
                out = work(k)
                s.synchronize()
                if not _same(torch, out, ref[k]):
                    bad.append(k)

    ts = [threading.Thread(target=run, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_streams_that_come_and_go(case):
    torch, G, work, ref = case
    note("workspace: destroyed streams")
    hip = ctypes.CDLL("libamdhip64.so")
    for k in range(8):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        out = work(k % 4, stream=s.value)
        # destroyed with its work pending; the next stream may get its address
        assert hip.hipStreamDestroy(s) == 0
        nxt = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(nxt), 1) == 0
        out2 = work((k + 1) % 4, stream=nxt.value)
        torch.cuda.synchronize()
        assert _same(torch, out, ref[k % 4]) and _same(torch, out2, ref[(k + 1) % 4])
        assert hip.hipStreamDestroy(nxt) == 0


def test_more_than_is_kept(case):
    torch, G, work, ref = case
    note("workspace: many sizes, then a graph freed")
    for n in range(100000, 1100000, 130000):
        g = G.gcn_build_csr(n, n, torch.arange(n, dtype=torch.int32, device="cuda:0"),
                            torch.zeros(n, dtype=torch.int32, device="cuda:0"), 0)
        Y = G.gcn_aggregate_fwd(g, torch.ones(n, 8, device="cuda:0"))
        assert Y[0, 0].item() == n and Y[1:].abs().max().item() == 0
        g.free()
    torch.cuda.synchronize()
    assert _same(torch, work(0), ref[0])


def test_blocks_past_the_limit_go_while_their_work_is_pending(case):
    torch, G, work, ref = case
    note("workspace: a limit of 1 MiB")
    tiny = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    old = os.environ.get("GCN_IDLE_MAX")
    os.environ["GCN_IDLE_MAX"] = str(1 << 20)
    try:
        G.gcn_build_csr(1, 1, tiny, tiny, 0).free()  # the limit is read with a graph
        streams = [torch.cuda.Stream() for _ in range(2)]
        torch.cuda.synchronize()
        out = []
        for rep in range(6):  # no waiting between the calls
            for k, s in enumerate(streams):
                with torch.cuda.stream(s):
                    out.append((k, work(k)))
            out.append((2, work(2)))
        torch.cuda.synchronize()
        assert all(_same(torch, y, ref[k]) for k, y in out)
    finally:
        if old is None:
            del os.environ["GCN_IDLE_MAX"]
        else:
            os.environ["GCN_IDLE_MAX"] = old
        G.gcn_build_csr(1, 1, tiny, tiny, 0).free()
