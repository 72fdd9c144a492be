"""The calls whose speed matters to a user of this library, over their sizes.

A case is a dict of plain values; its "kind" names the call sequence:

  aggregate   forward and transposed aggregation of a normalized graph
  halo        the same passes with the last quarter of the input rows held as
              8-bit or 2-bit codes (one worker's view of its boundary rows)
  exchange    one layer's quantized exchange on a partition: the sender's
              LayerNorm + quantize, the receiver's aggregation of local and
              received rows with the received partial sums added, and the
              transposed aggregation of the backward pass
  build       graph construction, normalization and the first aggregations
  dense       a class layer out of single calls: LayerNorm, product, softmax
              cross-entropy, both gradient products, LayerNorm backward
  gcn2        one training step of the 2-layer GCN
  sage3       one training step of the 3-layer GraphSAGE model with label
              propagation, and its forward pass for the logits

Graphs are RMAT (quadrants .57/.19/.19/.05, relabelled by a permutation) or
uniform; every input is drawn on the GPU from the seed.
"""

import math

import torch

import paper_2411_16025_amd as gcn

DEV = "cuda"


def listed():
    return [
        # A graph of a few thousand nodes, all of it in the caches: sampled
        # subgraphs and the unit of a serving loop. Launches and latency count.
        dict(name="agg_er4096_f64", kind="aggregate", graph="uniform", n=4096, draws=65536,
             f=64, dtype="f32"),
        # A citation-graph size with bf16 features at the hidden width.
        dict(name="agg_170k_f256_bf16", kind="aggregate", graph="rmat", n=170003, draws=1190021,
             f=256, dtype="bf16"),
        # The mid-size power-law graph of the benchmark.
        dict(name="agg_rmat20_f128", kind="aggregate", graph="rmat", n=1 << 20, draws=16 << 20,
             f=128, dtype="f32"),
        # The product-shaped graph at the class width: 47 contiguous columns.
        dict(name="agg_product_f47", kind="aggregate", graph="rmat", n=2449029, draws=65794508,
             f=47, dtype="f32"),
        # The benchmark's default workload: 2^24 nodes, a quarter of the input
        # rows received as 8-bit codes.
        dict(name="halo8_rmat24_f128", kind="halo", n=1 << 24, draws=32 << 24, f=128, bits=8),
        # One worker's share of a partitioned graph with the 2-bit exchange.
        dict(name="exchange2_partition_f128", kind="exchange", n_local=3500000, n_halo=1500000,
             draws=38000000, f=128, bits=2),
        # What every program pays once per graph before its first epoch.
        dict(name="build_rmat20", kind="build", n=1 << 20, draws=16 << 20, f=100, directed=False),
        # The class layer of the GraphSAGE model out of its single calls.
        dict(name="dense_500k_256_47", kind="dense", n=500000, f=256, classes=47),
        # A training step whose kernels are all short: the small end of a sweep.
        dict(name="gcn2_3k", kind="gcn2", n=3000, draws=24000, f=100, hidden=64, classes=10),
        # The training steps of the benchmark on the product-shaped graph.
        dict(name="gcn2_product", kind="gcn2", n=2449029, draws=65794508, f=100, hidden=256,
             classes=47),
        dict(name="sage3_170k", kind="sage3", n=170003, draws=1190021, f=128, hidden=256,
             classes=40),
        dict(name="sage3_product", kind="sage3", n=2449029, draws=65794508, f=100, hidden=256,
             classes=47),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["aggregate", "aggregate", "halo", "exchange", "build", "dense", "gcn2",
                       "sage3"])
    if kind == "aggregate":
        n = _log(rng, 4096, 2449029)
        f = rng.choice([_log(rng, 16, 256), 4 * _log(rng, 4, 64), rng.choice([47, 64, 100, 128, 256])])
        return dict(kind=kind, graph=rng.choice(["rmat", "rmat", "uniform"]), n=n,
                    draws=n * rng.randint(6, 27), f=f, dtype=rng.choice(["f32", "f32", "bf16"]))
    if kind == "halo":
        n = _log(rng, 1 << 16, 1 << 23)
        return dict(kind=kind, n=n, draws=n * rng.randint(8, 32),
                    f=rng.choice([64, 100, 128, 128, 256]), bits=rng.choice([8, 2]))
    if kind == "exchange":
        n = _log(rng, 40000, 3500000)
        return dict(kind=kind, n_local=n, n_halo=int(n * rng.uniform(0.2, 0.5)),
                    draws=n * rng.randint(6, 11), f=rng.choice([64, 100, 128, 256]),
                    bits=rng.choice([8, 2]))
    if kind == "build":
        n = _log(rng, 4096, 1 << 20)
        return dict(kind=kind, n=n, draws=n * rng.randint(6, 16), f=rng.choice([47, 64, 100, 128]),
                    directed=rng.random() < 0.5)
    if kind == "dense":
        return dict(kind=kind, n=_log(rng, 4096, 1000000), f=rng.choice([64, 100, 128, 256]),
                    classes=rng.randint(2, 64))
    n = _log(rng, 1000, 1000000)
    return dict(kind=kind, n=n, draws=n * rng.randint(5, 26), f=rng.choice([47, 64, 100, 128]),
                hidden=rng.choice([64, 100, 128, 256]), classes=rng.randint(5, 64))


# ---- inputs --------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform_pairs(n, m, g):
    e = torch.randint(0, n, (2, m), generator=g, device=DEV, dtype=torch.int32)
    return e[0].contiguous(), e[1].contiguous()


def _rmat_pairs(n, m, g):
    """m RMAT draws over [0, n) (rejected from the next power of two),
    relabelled by a random permutation."""
    bits = max(1, (n - 1).bit_length())
    perm = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
    us = torch.empty(m, dtype=torch.int32, device=DEV)
    vs = torch.empty(m, dtype=torch.int32, device=DEV)
    have = 0
    while have < m:
        k = min(1 << 26, int(1.5 * (m - have)) + 1024)
        u = torch.zeros(k, dtype=torch.int32, device=DEV)
        v = torch.zeros(k, dtype=torch.int32, device=DEV)
        for _ in range(bits):
            r = torch.rand(k, generator=g, device=DEV)
            low = r >= 0.76
            u.mul_(2).add_(low)
            v.mul_(2).add_(((r >= 0.57) & ~low) | (r >= 0.95))
        if n != 1 << bits:
            keep = (u < n) & (v < n)
            u, v = u[keep], v[keep]
        t = min(u.numel(), m - have)
        us[have:have + t] = perm.index_select(0, u[:t])
        vs[have:have + t] = perm.index_select(0, v[:t])
        have += t
    return us, vs


def _pairs(case, g):
    if case.get("graph") == "uniform":
        return _uniform_pairs(case["n"], case["draws"], g)
    return _rmat_pairs(case["n"], case["draws"], g)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _glorot(g, a, b):
    return (torch.rand(a, b, generator=g, device=DEV) * 2 - 1) * math.sqrt(6.0 / (a + b))


def _codes(x, bits):
    """Per-row codes (2-bit packed four per byte) and (zero point, scale)
    pairs of fp32 rows."""
    top = (1 << bits) - 1
    z = x.amin(1)
    s = (x.amax(1) - z) / top
    q = ((x - z[:, None]) / s[:, None]).round_().clamp_(0, top).to(torch.uint8)
    if bits == 2:
        pad = -q.shape[1] % 4
        q = torch.nn.functional.pad(q, (0, pad)).view(q.shape[0], -1, 4)
        q = (q[..., 0] | (q[..., 1] << 2) | (q[..., 2] << 4) | (q[..., 3] << 6)).contiguous()
    return q, torch.stack([z, s], 1).contiguous()


def _decode(q, zs, bits, f):
    """The float64 values of _codes' rows."""
    if bits == 2:
        q = torch.stack([(q >> s) & 3 for s in (0, 2, 4, 6)], 2).reshape(q.shape[0], -1)[:, :f]
    return q.double() * zs[:, 1:].double() + zs[:, :1].double()


def _partition(case, g):
    """(src, dst, deg) of one worker's rows: every pair with a local end adds
    the entry of that end's row; deg stands in for the degrees in the whole graph."""
    n_loc, n = case["n_local"], case["n_local"] + case["n_halo"]
    u, v = _rmat_pairs(n, case["draws"], g)
    a, b = v < n_loc, u < n_loc
    src, dst = torch.cat([u[a], v[b]]), torch.cat([v[a], u[b]])
    deg = torch.bincount(u, minlength=n) + torch.bincount(v, minlength=n)
    return src, dst, (deg * 2.2).to(torch.int32)


def _raw(case, seed):
    """The inputs of a case as torch tensors, from the seed alone."""
    g = _gen(seed)
    kind, f = case["kind"], case["f"]
    d = dict(case=case)
    if kind == "dense":
        n, c = case["n"], case["classes"]
        d["H"] = _normal(g, n, f).clamp_(min=0)  # a ReLU output
        d["W"] = _glorot(g, f, c)
        d["labels"] = torch.randint(0, c, (n,), generator=g, device=DEV, dtype=torch.int32)
        return d
    if kind == "exchange":
        n_loc, n_halo = case["n_local"], case["n_halo"]
        d["src"], d["dst"], d["deg"] = _partition(case, g)
        d["X"] = _normal(g, n_loc, f)
        d["B"] = _normal(g, n_halo, f)  # the boundary rows, as their owner holds them
        d["G"] = _normal(g, n_loc, f)
        n_part = max(1, n_halo // 8)  # partial sums received for as many local rows
        d["P"] = _normal(g, n_part, f)
        d["idx"] = torch.randperm(n_loc, generator=g, device=DEV)[:n_part].to(torch.int32)
        return d
    n = case["n"]
    d["src"], d["dst"] = _pairs(case, g)
    if kind in ("aggregate", "build"):
        d["X"] = _normal(g, n, f)
        d["G"] = _normal(g, n, f)
        if case.get("dtype") == "bf16":
            d["X"], d["G"] = d["X"].bfloat16(), d["G"].bfloat16()
    elif kind == "halo":
        n_loc = n - n // 4
        for x, q in (("X", "QX"), ("G", "QG")):
            t = _normal(g, n, f)
            d[q], d[q + "_zs"] = _codes(t[n_loc:], case["bits"])
            d[x] = t[:n_loc].clone()
            del t
    else:
        c, h = case["classes"], case["hidden"]
        d["X"] = _normal(g, n, f)
        d["labels"] = torch.randint(0, c, (n,), generator=g, device=DEV, dtype=torch.int32)
        if kind == "gcn2":
            d["W"] = [_glorot(g, f, h), _glorot(g, h, c)]
        else:
            d["W"] = []
            for a, b in ((f, h), (h, h), (h, c)):
                d["W"] += [_glorot(g, a, b), _glorot(g, a, b),
                           (torch.rand(b, generator=g, device=DEV) * 2 - 1) * 0.1]
            d["E"] = _glorot(g, c, f)
            d["mask"] = (torch.rand(n, generator=g, device=DEV) < 0.5).to(torch.uint8)
    return d


def _flags(case):
    if case["kind"] == "sage3":
        return gcn.GCN_SYMMETRIZE
    if case["kind"] == "exchange" or case.get("directed"):
        return gcn.GCN_ADD_SELF_LOOPS
    return gcn.GCN_SYMMETRIZE | gcn.GCN_ADD_SELF_LOOPS


def prepare(case, seed):
    s = _raw(case, seed)
    kind = case["kind"]
    if kind in ("dense", "build"):
        return s
    if kind == "exchange":
        n_loc = case["n_local"]
        s["graph"] = gcn.gcn_build_csr(n_loc, n_loc + case["n_halo"], s.pop("src"), s.pop("dst"),
                                       _flags(case))
        gcn.gcn_normalize(s["graph"], s.pop("deg"))
        s["Q"], s["zmin"], s["scale"] = gcn.gcn_layernorm_quantize(s.pop("P"), bits=case["bits"],
                                                                   layernorm=False)
        return s
    s["graph"] = gcn.gcn_build_csr(case["n"], case["n"], s.pop("src"), s.pop("dst"), _flags(case))
    if kind == "sage3":
        gcn.gcn_normalize_mean(s["graph"])
    else:
        gcn.gcn_normalize(s["graph"])
    return s


# ---- one pass -------------------------------------------------------------------


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "aggregate":
        return (gcn.gcn_aggregate_fwd(s["graph"], s["X"]), gcn.gcn_aggregate_bwd(s["graph"], s["G"]))
    if kind == "halo":
        out = []
        for x, q, csc in (("X", "QX", False), ("G", "QG", True)):
            zs = s[q + "_zs"]
            out.append(gcn.gcn_aggregate_fwd_q8halo(s["graph"], s[x].shape[0], s[x], s[q],
                                                    zs[:, 0], zs[:, 1], use_csc=csc, F=case["f"],
                                                    bits=case["bits"]))
        return tuple(out)
    if kind == "exchange":
        bits = case["bits"]
        q, zmin, scale = gcn.gcn_layernorm_quantize(s["B"], bits=bits)
        y = gcn.gcn_aggregate_fwd_q8halo(s["graph"], case["n_local"], s["X"], q, zmin, scale,
                                         bits=bits)
        gcn.gcn_add_rows_q(s["Q"], s["zmin"], s["scale"], s["idx"], y, bits=bits)
        return dict(q=q, zmin=zmin, scale=scale, y=y, dx=gcn.gcn_aggregate_bwd(s["graph"], s["G"]))
    if kind == "build":
        n = case["n"]
        g = gcn.gcn_build_csr(n, n, s["src"], s["dst"], _flags(case))
        gcn.gcn_normalize(g)
        s["graph"] = g  # kept by the program for its epochs
        return gcn.gcn_aggregate_fwd(g, s["X"]), gcn.gcn_aggregate_bwd(g, s["G"])
    if kind == "dense":
        y, rstd = gcn.gcn_layernorm_fwd(s["H"])
        z = gcn.gcn_gemm_f32(gcn.GCN_GEMM_NN, y, s["W"])
        loss, dz = gcn.gcn_softmax_xent(z, s["labels"])
        dw = gcn.gcn_gemm_f32(gcn.GCN_GEMM_TN, y, dz)
        dy = gcn.gcn_gemm_f32(gcn.GCN_GEMM_NT, dz, s["W"])
        return dict(y=y, z=z, loss=loss, dz=dz, dw=dw, dh=gcn.gcn_layernorm_bwd(y, rstd, dy,
                                                                             mask=s["H"]))
    if kind == "gcn2":
        return gcn.gcn_gcn2_step(s["graph"], s["X"], s["W"][0], s["W"][1], s["labels"])
    loss, grads, de = gcn.gcn_sage3_step(s["graph"], s["X"], s["W"], s["labels"], s["mask"], s["E"])
    logits = gcn.gcn_sage3_forward(s["graph"], s["X"], s["W"], s["labels"], s["mask"], s["E"])[2]
    return dict(loss=loss, grads=grads, de=de, logits=logits)


# ---- what a pass cannot do without ----------------------------------------------


def work(case):
    kind, f = case["kind"], case["f"]
    if kind == "dense":
        n, c = case["n"], case["classes"]
        # H, the labels and W in; y, z, dz, dh and dw out
        return dict(bytes=4.0 * (n * (3 * f + 2 * c + 1) + 2 * f * c), flops=6.0 * n * f * c)
    if kind == "exchange":
        n_loc, n_halo = case["n_local"], case["n_halo"]
        share = n_loc / (n_loc + n_halo)
        nnz = 2.0 * case["draws"] * share + n_loc
        row = f * case["bits"] / 8 + 8
        n_part = max(1, n_halo // 8)
        b = n_halo * (4.0 * f + row) + n_loc * 12.0 * f + n_part * row + (n_loc + n_halo) * 4.0 * f
        return dict(bytes=b + 16.0 * nnz, flops=4.0 * nnz * f)
    n, m = case["n"], case["draws"]
    nnz = float(m + n if case.get("directed") else 2 * m + n)
    if kind == "sage3":
        nnz -= n
    if kind in ("aggregate", "build"):
        e = 2 if case.get("dtype") == "bf16" else 4
        b = 16.0 * nnz + 2.0 * n * f * (4 + e)
        if kind == "build":
            b += 8.0 * m + 16.0 * nnz * (2 if case["directed"] else 1)  # pairs in, (column, value) out
        return dict(bytes=b, flops=4.0 * nnz * f)
    if kind == "halo":
        row = 0.75 * 4.0 * f + 0.25 * (f * case["bits"] / 8 + 8)
        return dict(bytes=2.0 * (8.0 * nnz + n * (row + 4.0 * f)), flops=4.0 * nnz * f)
    h, c = case["hidden"], case["classes"]
    if kind == "gcn2":
        lo = min(f, h)
        agg = lo + 2 * c + (0 if f <= h else h)
        return dict(bytes=4.0 * n * f + 8.0 * nnz + 8.0 * (f * h + h * c),
                    flops=2.0 * nnz * agg + 2.0 * n * (2 * f * h + 3 * h * c))
    w = 2 * (f * h + h * h + h * c)
    # step: forward and twice its products backward; forward once more; the
    # aggregations at the narrower width of each layer
    agg = 2 * (min(f, h) + h + min(h, c)) + min(f, h) + h + min(h, c)
    return dict(bytes=2 * (4.0 * n * f + 8.0 * nnz) + 4.0 * (4 * w + n * c),
                flops=2.0 * nnz * agg + 2.0 * n * w * 4)


def tolerance(case):
    # 32-bit sums in any order: aggregations are within 1.3e-7 of the same sums
    # in 64 bits, the products of a layer within 3e-7. Whole values are codes,
    # which a last bit of a LayerNorm moves at the half steps between two
    # codes (and with them the rows that gather them). A training step passes
    # a unit's gradient or not by the sign of a sum: the units whose sum rounds
    # to the other side of 0 move its gradients by 2e-4, or by 2e-3 where a
    # single one of 3,000 x 64 units does.
    kind = case["kind"]
    if kind in ("gcn2", "sage3"):
        return dict(rel=2e-3, max=0.5)
    if kind == "exchange":
        return dict(rel=1e-4, max=0.5, differ=1e-5)
    return dict(rel=2e-6 if kind == "dense" else 1e-6)


# ---- the same in 64 bits ---------------------------------------------------------


class _Sparse:
    """Entries (row, col) of the stored matrix, sorted and distinct."""

    def __init__(self, case, d):
        flags = _flags(case)
        n_rows = case.get("n", case.get("n_local"))
        n_cols = n_rows + case.get("n_halo", 0)
        src, dst = d["src"].long(), d["dst"].long()
        if flags & gcn.GCN_ADD_SELF_LOOPS:
            keep = src != dst
            src, dst = src[keep], dst[keep]
        keys = dst * n_cols + src
        if flags & gcn.GCN_SYMMETRIZE:
            keys = torch.cat([keys, src * n_cols + dst])
        if flags & gcn.GCN_ADD_SELF_LOOPS:
            i = torch.arange(min(n_rows, n_cols), device=DEV)
            keys = torch.cat([keys, i * n_cols + i])
        del src, dst
        keys = torch.unique(keys)
        self.row, self.col = keys // n_cols, keys % n_cols
        self.n_rows, self.n_cols = n_rows, n_cols
        length = torch.bincount(self.row, minlength=n_rows)
        if case["kind"] == "sage3":
            self.val = 1.0 / length.double()[self.row]
            return
        if "deg" in d:
            deg = d["deg"].long()
        else:
            deg = length - torch.bincount(self.row[self.row == self.col], minlength=n_rows)
        t = deg.double() + 1
        self.val = 1.0 / torch.sqrt(t[self.row] * t[self.col])

    def mm(self, x, transposed=False):
        a, b = (self.col, self.row) if transposed else (self.row, self.col)
        x = x.double()
        y = torch.zeros(self.n_cols if transposed else self.n_rows, x.shape[1],
                        dtype=torch.float64, device=DEV)
        step = max(1, (1 << 28) // x.shape[1])
        for i in range(0, a.numel(), step):
            j = slice(i, i + step)
            y.index_add_(0, a[j], x.index_select(0, b[j]).mul_(self.val[j, None]))
        return y


def _norm64(x):
    x = x.double()
    d = x - x.mean(1, keepdim=True)
    rstd = 1.0 / torch.sqrt((d * d).mean(1, keepdim=True) + 1e-5)
    return d * rstd, rstd


def _norm_back64(y, rstd, g):
    return rstd * (g - g.mean(1, keepdim=True) - y * (g * y).mean(1, keepdim=True))


def _xent64(z, labels, keep=None):
    p = torch.log_softmax(z, 1)
    i = torch.arange(z.shape[0], device=DEV)
    hit = p[i, labels.long()]
    keep = torch.ones_like(hit) if keep is None else keep.double()
    n = keep.sum().clamp(min=1)
    g = p.exp()
    g[i, labels.long()] -= 1
    return -(hit * keep).sum() / n, g * (keep / n)[:, None]


def _t(x):
    return x.t().contiguous()


def _gcn64(a, d):
    w1, w2 = (w.double() for w in d["W"])
    p = a.mm(d["X"])
    h = (p @ w1).clamp_(min=0)
    loss, dl = _xent64(a.mm(h @ w2), d["labels"])
    dz2 = a.mm(dl, True)
    dz1 = (dz2 @ _t(w2)) * (h > 0)
    return loss, _t(p) @ dz1, _t(h) @ dz2


def _sage64(a, d):
    w = [t.double() for t in d["W"]]
    mask = d["mask"].bool()
    x = d["X"].double()
    x[mask] += d["E"].double()[d["labels"].long()[mask]]
    h, kept = x, []
    for l in range(3):
        y, rstd = _norm64(h)
        z = a.mm(y)
        o = y @ w[3 * l] + z @ w[3 * l + 1] + w[3 * l + 2]
        kept.append((y, rstd, z))
        h = o.clamp(min=0) if l < 2 else o
        kept[-1] += (h,)
    loss, do = _xent64(h, d["labels"], ~mask)
    grads = [None] * 9
    for l in (2, 1, 0):
        y, rstd, z, _ = kept[l]
        grads[3 * l:3 * l + 3] = [_t(y) @ do, _t(z) @ do, do.sum(0)]
        dy = do @ _t(w[3 * l]) + a.mm(do @ _t(w[3 * l + 1]), True)
        do = _norm_back64(y, rstd, dy)
        if l > 0:
            do *= kept[l - 1][3] > 0
    de = torch.zeros_like(d["E"], dtype=torch.float64)
    de.index_add_(0, d["labels"].long()[mask], do[mask])
    return dict(loss=loss, grads=grads, de=de, logits=h)


def exact(case, seed):
    kind = case["kind"]
    if case.get("draws", 0) > 1 << 27:
        return None  # the billion entries of the largest graph take too long
    d = _raw(case, seed)
    if kind == "dense":
        y, rstd = _norm64(d["H"])
        w = d["W"].double()
        z = y @ w
        loss, dz = _xent64(z, d["labels"])
        dh = _norm_back64(y, rstd, dz @ _t(w)) * (d["H"] > 0)
        return dict(y=y, z=z, loss=loss, dz=dz, dw=_t(y) @ dz, dh=dh)
    a = _Sparse(case, d)
    if kind in ("aggregate", "build"):
        return a.mm(d["X"]), a.mm(d["G"], True)
    if kind == "halo":
        out = []
        for x, q, csc in (("X", "QX", False), ("G", "QG", True)):
            full = torch.cat([d[x].double(), _decode(d[q], d[q + "_zs"], case["bits"], case["f"])])
            out.append(a.mm(full, csc))
        return tuple(out)
    if kind == "exchange":
        y = _norm64(d["B"])[0]
        zmin = y.amin(1)
        # y follows rounded codes: no value of its own in 64 bits
        return dict(q=None, zmin=zmin, scale=(y.amax(1) - zmin) / ((1 << case["bits"]) - 1), y=None,
                    dx=a.mm(d["G"], True))
    return _gcn64(a, d) if kind == "gcn2" else _sage64(a, d)
