"""GPU parity of the fp32 products on the bf16 matrix cores.

Against float64 products of the same inputs, within 1e-5 of the sum of |terms|
per element (a sum of K <= 4096 terms with one rounding per 16 of each of six
part products is within 6 K / 16 * 2^-24 <= 9.2e-5 at the very worst, and
rounding errors of either sign leave a few 1e-7), on both sides of the column,
row and K tiles; and infinities and NaN where an fp32 product has them. The masked and ReLU products,
which only the training steps form, through the GCN step.
"""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_close, dev, host, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2411_16025_amd as pkg
    pkg.lib()
    return pkg


def _pair(A, B):
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    return A64 @ B64, np.abs(A64) @ np.abs(B64)


# contiguous operands of odd widths (every load 4-byte aligned), 1 to 9 column
# blocks of 32, K around the 16-deep step, rows around the 64-, 128- and
# 256-row tiles; the aligned ones are large enough to leave the general tile
TALL = [(4096, 2, 17), (4097, 33, 16), (4223, 47, 256), (5000, 65, 31), (4096, 97, 33),
        (4100, 161, 47), (4099, 255, 19), (4161, 257, 63), (32769, 301, 21), (33023, 256, 200),
        (70001, 100, 256), (16448, 200, 516)]


@pytest.mark.parametrize("M,N,K", TALL)
def test_tall(G, M, N, K):
    import torch
    note("split tall %dx%dx%d" % (M, N, K))
    A, B = synth.uniform(301, M, K), synth.uniform(302, K, N)
    ref, S = _pair(A, B)
    C = torch.full((M, N + 3), 7.0, device="cuda:0")
    out = G.gcn_gemm_f32(G.GCN_GEMM_NN, dev(A), dev(B), C=C[:, :N])
    assert_close(host(out), ref, S, what="NN")
    assert np.all(host(C)[:, N:] == 7.0)
    again = G.gcn_gemm_f32(G.GCN_GEMM_NN, dev(A), dev(B))
    assert torch.equal(again.view(torch.int32), out.contiguous().view(torch.int32))
    out = G.gcn_gemm_f32(G.GCN_GEMM_NT, dev(A), dev(np.ascontiguousarray(B.T)))
    assert_close(host(out), ref, S, what="NT")


# every tile width, one and several chunks, partial steps, an odd and an even
# number of chunks (the sign alternates), both tile sizes of wide outputs
TN = [(64, 1, 1), (255, 33, 31), (257, 129, 32), (1000, 47, 33), (4111, 128, 64), (4111, 100, 65),
      (20000, 257, 129), (9999, 16, 300), (131073, 129, 130), (140001, 300, 257)]


@pytest.mark.parametrize("K,M,N", TN)
def test_tn(G, K, M, N):
    import torch
    note("split tn %dx%dx%d" % (K, M, N))
    A, B = synth.uniform(303, K, M), synth.uniform(304, K, N)
    ref, S = _pair(np.ascontiguousarray(A.T), B)
    C = G.gcn_gemm_f32(G.GCN_GEMM_TN, dev(A), dev(B))
    assert_close(host(C), ref, S, what="TN")
    C2 = G.gcn_gemm_f32(G.GCN_GEMM_TN, dev(A), dev(B))
    assert torch.equal(C.view(torch.int32), C2.view(torch.int32))


def test_bias_cancels_over_rows(G):
    """Column sums of a product of a million rows: a rounding of one sign in
    every element would add up (2e-9 of an element's size, a million times)."""
    import torch
    note("split bias")
    A = torch.randn(1 << 20, 128, device="cuda:0")
    B = torch.randn(128, 128, device="cuda:0")
    C = G.gcn_gemm_f32(G.GCN_GEMM_NN, A, B)
    err = (C.double() - A.double() @ B.double()).sum(0)
    # 2^20 independent errors of about 2.5e-7 * sqrt(128) each: 3e-3; six deviations
    assert err.abs().max().item() < 6 * 1024 * 2.5e-7 * 128 ** 0.5


@pytest.mark.parametrize("op", ["NN", "NT", "TN"])
def test_not_finite(G, op):
    import torch
    note("split not finite %s" % op)
    M, N, K = (5000, 47, 33) if op != "TN" else (40, 47, 5000)
    A, B = synth.uniform(305, M, K), synth.uniform(306, K, N)
    A[3, 5] = np.inf
    A[17, 2] = np.nan
    A[39, 7] = 3.4e38   # rounds up to infinity in bf16
    B[7, 1] = 0.5
    B[7, 2] = 8.0       # overflows
    B[5, 4] = 0.0       # inf * 0
    with np.errstate(all="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64)
        want = ref.astype(np.float32)
    if op == "TN":
        C = G.gcn_gemm_f32(G.GCN_GEMM_TN, dev(np.ascontiguousarray(A.T)), dev(B))
    elif op == "NT":
        C = G.gcn_gemm_f32(G.GCN_GEMM_NT, dev(A), dev(np.ascontiguousarray(B.T)))
    else:
        C = G.gcn_gemm_f32(G.GCN_GEMM_NN, dev(A), dev(B))
    got = host(C)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isinf(got), np.isinf(want))
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf])
    fin = np.isfinite(want)
    scale = np.nan_to_num(np.abs(A), nan=0, posinf=0).astype(np.float64) @ np.abs(B).astype(np.float64)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-5 * scale[fin])


@pytest.mark.parametrize("op,M,N,K", [("NN", 4097, 47, 100), ("NN", 8192, 256, 100),
                                      ("NT", 4100, 161, 47)])
def test_captured(G, op, M, N, K):
    """Captured products record kernels only (no allocation), and every replay
    multiplies what the operands hold then."""
    import torch
    note("split captured %s %s" % (op, (M, N, K)))
    code = G.GCN_GEMM_NN if op == "NN" else G.GCN_GEMM_NT
    Ad, Bd = torch.empty((M, K), device="cuda:0"), torch.empty(
        (K, N) if op == "NN" else (N, K), device="cuda:0")
    Cd = torch.empty((M, N), device="cuda:0")
    Ad.fill_(1.0)
    Bd.fill_(1.0)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()  # default priority
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        G.gcn_gemm_f32(code, Ad, Bd, C=Cd)
    torch.cuda.synchronize()
    for rep in range(3):
        A, B = synth.uniform(310 + rep, M, K), synth.uniform(320 + rep, K, N)
        Ad.copy_(dev(A))
        Bd.copy_(dev(B if op == "NN" else np.ascontiguousarray(B.T)))
        Cd.fill_(7.0)  # eager work between the replays
        eager = host(G.gcn_gemm_f32(code, Ad, Bd))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want, scale = _pair(A, B)
        assert_close(host(Cd), want, scale, what="replay %d" % rep)
        assert_close(eager, want, scale, what="eager %d" % rep)


@pytest.mark.parametrize("op,M,N,K", [("NN", 4097, 47, 100), ("NN", 40000, 256, 101),
                                      ("NN", 5000, 192, 516), ("NT", 40000, 200, 128),
                                      ("NT", 4100, 161, 47)])
def test_captured_bits(G, op, M, N, K):
    """A captured product is the eager one, bit for bit."""
    import torch
    note("split captured bits %s %s" % (op, (M, N, K)))
    code = G.GCN_GEMM_NN if op == "NN" else G.GCN_GEMM_NT
    Ad = torch.zeros((M, K), device="cuda:0")
    Bd = dev(synth.uniform(341, K, N) if op == "NN" else synth.uniform(341, N, K))
    Cd = torch.empty((M, N), device="cuda:0")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()  # default priority
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        G.gcn_gemm_f32(code, Ad, Bd, C=Cd)
    torch.cuda.synchronize()
    for rep in range(3):
        Ad.copy_(dev(synth.uniform(342 + rep, M, K)))
        Cd.fill_(7.0)  # eager work between the replays
        eager = G.gcn_gemm_f32(code, Ad, Bd)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(eager.view(torch.int32), Cd.view(torch.int32))


# B is split by every workgroup: its units over the threads of each tile width,
# rows and columns past its edges, both ways it can be stored
@pytest.mark.parametrize("M,N,K", [(4096, 31, 16), (4099, 63, 18), (4096, 128, 33), (4100, 191, 31),
                                   (4100, 193, 47), (33000, 225, 30), (40000, 449, 65)])
def test_b_edges(G, M, N, K):
    import torch
    note("split B edges %dx%dx%d" % (M, N, K))
    A, B = synth.uniform(351, M, K + 1)[:, :K], synth.uniform(352, K, N)
    ref, S = _pair(A, B)
    for ld in (N, N + 5):  # rows of B, then of its transpose, inside wider ones
        Bp = torch.full((K, ld), float("nan"), device="cuda:0")
        Bp[:, :N] = dev(B)
        out = G.gcn_gemm_f32(G.GCN_GEMM_NN, dev(np.ascontiguousarray(A)), Bp[:, :N])
        assert_close(host(out), ref, S, what="NN")
        Bt = torch.full((N, K + ld - N), float("nan"), device="cuda:0")
        Bt[:, :K] = dev(np.ascontiguousarray(B.T))
        out = G.gcn_gemm_f32(G.GCN_GEMM_NT, dev(np.ascontiguousarray(A)), Bt[:, :K])
        assert_close(host(out), ref, S, what="NT")


# the tiles of every width, at their edges and inside, with a sum that is not
# finite: that tile is computed again, the others are not touched
@pytest.mark.parametrize("op,M,N,K", [("NN", 4100, 31, 19), ("NN", 4100, 64, 37), ("NN", 4100, 127, 40),
                                      ("NN", 33000, 192, 50), ("NN", 33000, 256, 96), ("NN", 5000, 255, 111),
                                      ("NT", 4100, 97, 36), ("NT", 33000, 256, 101), ("NT", 5000, 250, 259),
                                      ("TN", 300, 257, 131079), ("TN", 100, 100, 7003), ("TN", 40, 33, 2001),
                                      ("TN", 40, 20, 2001)])
def test_not_finite_tiles(G, op, M, N, K):
    import torch
    note("split not finite %s %s" % (op, (M, N, K)))
    gen = torch.Generator(device="cuda:0").manual_seed(360)
    A = torch.randn(M, K, device="cuda:0", generator=gen)
    B = torch.randn(K, N, device="cuda:0", generator=gen)
    ref, S = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    rows = {0: float("inf"), M // 2: float("nan"), M - 1: float("-inf")}
    for r, v in rows.items():
        A[r, K // 3] = v
    B[K // 3, N - 1] = 0.0
    if op == "TN":
        C = G.gcn_gemm_f32(G.GCN_GEMM_TN, A.t().contiguous(), B)
    elif op == "NT":
        C = G.gcn_gemm_f32(G.GCN_GEMM_NT, A, B.t().contiguous())
    else:
        C = G.gcn_gemm_f32(G.GCN_GEMM_NN, A, B)
    for r, v in rows.items():
        want = v * B[K // 3]  # infinities of either sign, NaN where B is 0
        assert torch.equal(torch.isnan(C[r]), torch.isnan(want))
        assert torch.equal(C[r].nan_to_num(nan=7.0), want.nan_to_num(nan=7.0))
    keep = torch.ones(M, dtype=torch.bool, device="cuda:0")
    keep[list(rows)] = False
    keep = keep[:, None] & (torch.arange(N, device="cuda:0") < N - 1)
    assert torch.all(((C.double() - ref).abs() <= 1e-5 * S)[keep])


def test_not_finite_time(G):
    """A diverged run's products take a few times as long, not a hundred (3.6
    times measured, 100 when the tiles were computed again element by element)."""
    import torch
    note("split not finite, time")
    A = torch.randn(32768, 516, device="cuda:0")
    B = torch.randn(516, 256, device="cuda:0")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def ms():
        best = float("inf")
        for _ in range(6):
            a.record()
            G.gcn_gemm_f32(G.GCN_GEMM_NN, A, B)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    finite = ms()
    A.fill_(float("nan"))
    assert ms() < 20 * finite


# fp32 holds 24 bits of a number down to 2^-126 and fewer below; so do the parts.
# Rounding errors of either sign leave 2.4e-7 here (2.9e-7 on the fp32
# instruction, which takes the largest numbers); four times that.
@pytest.mark.parametrize("ea,eb", [(0, 0), (-100, 20), (-112, 20), (-118, 20), (-124, 20), (-130, 20),
                                   (-140, 30), (20, -124), (60, -118), (-60, -55), (100, -60),
                                   (112, -100), (60, 40), (-100, 110)])
@pytest.mark.parametrize("op", ["NN", "NT", "TN"])
def test_range(G, op, ea, eb):
    import torch
    note("split operands of 2^%d and 2^%d, %s" % (ea, eb, op))
    gen = torch.Generator(device="cuda:0").manual_seed(370)
    M, N, K = (8000, 256, 256) if op != "TN" else (256, 128, 5000)
    A = torch.randn(M, K, device="cuda:0", generator=gen).double().mul(2.0 ** ea).float()
    B = torch.randn(K, N, device="cuda:0", generator=gen).double().mul(2.0 ** eb).float()
    ref = A.double() @ B.double()
    if op == "TN":
        C = G.gcn_gemm_f32(G.GCN_GEMM_TN, A.t().contiguous(), B)
    elif op == "NT":
        C = G.gcn_gemm_f32(G.GCN_GEMM_NT, A, B.t().contiguous())
    else:
        C = G.gcn_gemm_f32(G.GCN_GEMM_NN, A, B)
    rel = ((C.double() - ref).norm() / ref.norm()).item()
    note("rel %.2e" % rel)
    assert rel <= 1.2e-6


@pytest.mark.parametrize("K", [16, 100, 256, 1024])
def test_worst_operands(G, K):
    """All operands 1.0038834: the products left out are 2^-24 of each product,
    all of one sign. Beyond that a rounding per 16 of each of six products, at
    most 2^-24 of the sum each."""
    import torch
    note("split worst operands K=%d" % K)
    v = 1.0038834
    A = torch.full((32768, K), v, device="cuda:0")
    B = torch.full((K, 256), v, device="cuda:0")
    want = A[0, 0].double().item() ** 2
    bound = (1.001 + 6 * -(-K // 16)) * 2.0 ** -24
    nn = G.gcn_gemm_f32(G.GCN_GEMM_NN, A, B).double() / (want * K) - 1
    nt = G.gcn_gemm_f32(G.GCN_GEMM_NT, A, B.t().contiguous()).double() / (want * K) - 1
    note("NN %.2e NT %.2e" % (nn.abs().max(), nt.abs().max()))
    assert nn.abs().max() <= bound and nt.abs().max() <= bound
    A, B = torch.full((64 * K, 256), v, device="cuda:0"), torch.full((64 * K, 128), v, device="cuda:0")
    tn = G.gcn_gemm_f32(G.GCN_GEMM_TN, A, B).double() / (want * 64 * K) - 1
    note("TN %.2e" % tn.abs().max())
    assert tn.abs().max() <= (1.001 + 6 * 64 * K / 16) * 2.0 ** -24


@pytest.mark.parametrize("op", ["NN", "NT", "TN"])
def test_zero_sums_have_no_sign(G, op):
    """Sums of exact zeros are +0, as on the fp32 instruction, also where they are
    formed of negated products."""
    import torch
    note("split zeros %s" % op)
    M, N, K = (8000, 256, 256) if op != "TN" else (256, 128, 5000)
    A, B = torch.randn(M, K, device="cuda:0"), torch.randn(K, N, device="cuda:0")
    A[::3] = 0.0
    B[:, 5::7] = 0.0
    if op == "TN":
        C = G.gcn_gemm_f32(G.GCN_GEMM_TN, A.t().contiguous(), B)
    elif op == "NT":
        C = G.gcn_gemm_f32(G.GCN_GEMM_NT, A, B.t().contiguous())
    else:
        C = G.gcn_gemm_f32(G.GCN_GEMM_NN, A, B)
    bits = C.view(torch.int32)
    assert torch.all(bits[::3] == 0) and torch.all(bits[:, 5::7] == 0)


def _tn(M, N, K, seed):
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    A = torch.randn(K, M, device="cuda:0", generator=gen)
    B = torch.randn(K, N, device="cuda:0", generator=gen)
    ref = torch.zeros(M, N, device="cuda:0", dtype=torch.float64)
    for k in range(0, K, 1 << 18):
        ref += A[k:k + (1 << 18)].double().t().contiguous() @ B[k:k + (1 << 18)].double()
    return A, B, ref


# fp32 sums in chunks of 1024 rows leave 6.1e-7 (4 rows to a rounding); these
# no more, at the sizes whose chunks are longest
@pytest.mark.parametrize("M,N,K", [(512, 256, 500000), (300, 300, 500000), (1000, 1000, 20000),
                                   (1000, 520, 100001), (516, 256, 1000003)])
def test_tn_precision(G, M, N, K):
    note("split tn precision %dx%dx%d" % (M, N, K))
    A, B, ref = _tn(M, N, K, 380)
    C = G.gcn_gemm_f32(G.GCN_GEMM_TN, A, B)
    rel = ((C.double() - ref).norm() / ref.norm()).item()
    note("rel %.2e" % rel)
    assert rel <= 6.1e-7 if K < 1000000 else rel <= 8.7e-7  # 2048 rows there


def test_tn_partials(G):
    """Chunks that one workgroup adds up: the same bits every time, a chunk with an
    infinity among them, and the partial sums of no more than the fp32 kernel's
    (598 chunks of 4,096 rows) kept afterwards."""
    import torch
    note("split tn partials")
    M, N, K = 512, 256, 2449029
    A, B, ref = _tn(M, N, K, 381)
    C = torch.empty(M, N, device="cuda:0")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    G.gcn_gemm_f32(G.GCN_GEMM_TN, A, B, C=C)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] <= 1.3 * 598 * M * N * 4
    assert ((C.double() - ref).norm() / ref.norm()).item() <= 11.7e-7
    C2 = G.gcn_gemm_f32(G.GCN_GEMM_TN, A, B)
    assert torch.equal(C.view(torch.int32), C2.view(torch.int32))
    A[2000000, 7] = float("inf")
    C2 = G.gcn_gemm_f32(G.GCN_GEMM_TN, A, B)
    assert torch.equal(C2[7], float("inf") * B[2000000].sign())
    keep = torch.arange(M, device="cuda:0") != 7
    # (the tiles of that chunk are summed on the fp32 instruction)
    assert ((C2.double() - ref)[keep].norm() / ref[keep].norm()).item() <= 11.7e-7


# the unfused GCN step's dH1 = (dZ2 W2^T) masked (n x hidden x classes from 4e8 on) on
# each tile width, whole and cut tiles, and H1 = relu(P W1) where it aggregates first
@pytest.mark.parametrize("n,f_in,hidden,C", [(70001, 128, 128, 47), (100001, 132, 100, 47),
                                             (45001, 200, 192, 47), (34001, 128, 256, 47),
                                             (33001, 130, 250, 49)])
def test_masked_in_the_gcn_step(G, n, f_in, hidden, C):
    import torch
    assert n * hidden * C >= 4e8 and hidden > 64
    note("split masked, gcn step %s" % ((n, f_in, hidden, C),))
    src, dst = synth.rmat_edges(391, n, 4 * n, perm_seed=392)
    flags = synth.SYMMETRIZE | synth.ADD_SELF_LOOPS
    X, y = synth.normal(393, n, f_in), synth.labels(394, n, C)
    W1, W2 = synth.glorot(395, f_in, hidden), synth.glorot(396, hidden, C)
    g = G.gcn_build_csr(n, n, dev(src), dev(dst), flags)
    G.gcn_normalize(g)
    loss, dW1, dW2 = G.gcn_gcn2_step(g, dev(X), dev(W1), dev(W2), dev(y))
    torch.cuda.synchronize()
    g.free()
    og = oracle.Graph(n, n, src, dst, flags)
    ref = oracle.gcn_step(og, X, W1, W2, y)
    assert abs(float(loss) - ref["loss"]) <= 1e-5 * abs(ref["loss"])
    agg_t = lambda T: oracle._agg64(og.csc_ptr, og.csc_idx, og.csc_val, T)
    aX = np.abs(X).astype(np.float64)
    S1 = aX.T @ agg_t(np.abs(ref["dH1"]))
    S2 = np.abs(ref["H1"]).T @ agg_t(np.abs(ref["dlogits"]))
    # a unit whose sum is within fp32 rounding of 0 (2e-6 of its terms' magnitudes:
    # up to 200 products, then a row's entries) may pass its gradient or not
    agg = lambda T: oracle._agg64(og.csr_ptr, og.csr_idx, og.csr_val, T)
    near = np.abs(agg(X.astype(np.float64) @ W1)) <= 2e-6 * agg(aX @ np.abs(W1))
    note("%d units at 0" % near.sum())
    E1 = aX.T @ agg_t(np.abs(ref["dH1"]) * near)
    assert np.all(np.abs(host(dW1) - ref["dW1"]) <= 1e-5 * S1 + E1)
    assert_close(host(dW2), ref["dW2"], S2, what="dW2")
