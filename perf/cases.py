"""The work a user of this library has it do, as timed cases.

``listed()`` holds the fixed cases; ``draw(rng)`` one more of the same ranges.
A case is a dict of plain values; ``prepare`` makes its inputs on the GPU from
the seed, ``run`` takes them once through the public entry points, ``exact``
evaluates the same in float64 with plain torch, ``work`` counts the bytes and
operations that cannot be avoided.

Kinds of case
  gcn        two GCN layers (ReLU between), float32 or bfloat16; with
             ``plan`` the graph layout is part of the pass (a new graph each
             step), without it the plan is kept (a graph served many times)
  gat        two GAT layers (heads concatenated + ELU, then heads averaged)
  sage_pool  GraphSAGE-pool layer: Linear + ReLU, max over the in-edges,
             concat, Linear
  gated      gated edge-feature message passing with a GRU update (64 wide)
  sage_lstm  GraphSAGE layer with the LSTM Gather
  rgcn       R-GCN layer on typed edges; with ``plan`` everything from the raw
             CSR on (plan, typed layout, layer) is part of the pass
  plan       the layout of a graph that has just arrived, checked
  propagate  one fused Scatter + ApplyEdge + Gather with no weights (feature
             propagation, neighbour means and maxima)
  transform  one ApplyVertex product with its epilogue (the Linear of a layer
             that a program composes itself)

Graphs: "er" uniform pairs, "rmat" power law (a, b, c = 0.57, 0.19, 0.19,
relabelled), "ba" preferential attachment, "mesh" near neighbours on a torus
grid in random vertex order.  ``deg`` is the mean number of stored edges per
vertex before self-loops; ``loops`` adds one self-loop per vertex.
"""
import math

import torch

from paper_2009_00804_amd import layers as LY
from paper_2009_00804_amd import saga as S

DEV = "cuda"
BF16 = "bf16"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _case(kind, graph="er", v=0, deg=0, loops=False, dtype="f32", **kw):
    return dict(kind=kind, graph=graph, v=v, deg=deg, loops=loops, dtype=dtype, **kw)


def listed():
    return [
        # the smallest call: a citation-sized graph, where launches and latency count
        _case("gcn", "er", 2000, 5, True, f_in=128, hidden=16, f_out=8, plan=False, sparse=True,
              name="gcn_er_2k"),
        # the largest: a 2.1M-vertex power-law graph with 602 features, its plan in the step
        _case("gcn", "rmat", 1 << 21, 50, True, f_in=602, hidden=128, f_out=41, plan=True, sparse=False,
              name="gcn_rmat_2m"),
        # the same size served in bfloat16 on a plan that is kept
        _case("gcn", "rmat", 1 << 21, 50, True, BF16, f_in=602, hidden=128, f_out=41, plan=False,
              sparse=False, name="gcn_rmat_2m_bf16"),
        # attention on a mid-sized social graph: 8 heads x 8
        _case("gat", "ba", 20000, 10, True, f_in=512, heads=8, head_dim=8, name="gat_ba_20k"),
        # GraphSAGE-pool, 256 wide: two large products and a max over the in-edges
        _case("sage_pool", "rmat", 1 << 17, 16, f_in=256, f_out=256, name="sage_pool_rmat_131k"),
        # edge-feature message passing on a point cloud / molecule-like graph
        _case("gated", "mesh", 100000, 12, fe=16, name="gated_mesh_100k"),
        # the recurrence along every row's in-edges, hub rows included
        _case("sage_lstm", "rmat", 1 << 17, 16, f_in=256, hidden=128, f_out=256, name="sage_lstm_rmat_131k"),
        # typed edges, 32 relations, a kept layout
        _case("rgcn", "rmat", 1 << 18, 16, f_in=128, f_out=64, rels=32, plan=False, name="rgcn_rmat_262k"),
        # a typed graph that has just arrived: plan, typed layout and layer, bfloat16
        _case("rgcn", "rmat", 15000, 11, False, BF16, f_in=100, f_out=40, rels=9, plan=True,
              name="rgcn_new_15k_bf16"),
        # the layout alone, mid-sized uniform graph (what each sampled subgraph pays)
        _case("plan", "er", 100000, 12, True, name="plan_er_100k"),
        # neighbour means of raw features, an odd width, no weights
        _case("propagate", "rmat", 300000, 20, reduce="mean", norm=False, f_in=100,
              name="propagate_mean_300k"),
        # the concat Linear of a GraphSAGE layer in bfloat16, ragged in every size
        _case("transform", dtype=BF16, v=232965, k=300, k2=300, f_out=200, act="relu",
              name="transform_concat_bf16"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case, without a name."""
    kind = rng.choice(["gcn", "gcn", "gcn", "gat", "sage_pool", "gated", "sage_lstm", "rgcn", "rgcn", "plan",
                       "propagate", "propagate", "transform", "transform"])
    dtype = rng.choice(["f32", BF16])
    graph = rng.choice(["er", "rmat", "ba", "mesh"])
    loops = rng.random() < 0.5

    def size(lo, hi, deg_lo=2, deg_hi=50, edges=60_000_000):
        v = _logint(rng, lo, hi)
        deg = _logint(rng, deg_lo, min(deg_hi, v // 4))
        while v * deg > edges:
            deg = max(1, deg // 2)
        return v, deg + deg % 2  # "ba" and "mesh" store every edge in both directions

    if kind == "gcn":
        v, deg = size(500, 1 << 20)
        return _case(kind, graph, v, deg, loops, dtype, f_in=_logint(rng, 16, 602), hidden=_logint(rng, 8, 256),
                     f_out=_logint(rng, 3, 128), plan=rng.random() < 0.5, sparse=rng.random() < 0.2)
    if kind == "gat":
        v, deg = size(500, 200_000)
        heads, dim = rng.choice([(1, 16), (1, 64), (2, 32), (4, 8), (4, 16), (8, 4), (8, 8), (8, 16), (8, 32)])
        return _case(kind, graph, v, deg, True, f_in=_logint(rng, 16, 602), heads=heads, head_dim=dim)
    if kind == "sage_pool":
        v, deg = size(1000, 1 << 18)
        return _case(kind, graph, v, deg, loops, f_in=_logint(rng, 24, 512), f_out=_logint(rng, 8, 512))
    if kind == "gated":
        v, deg = size(1000, 300_000, 4, 24)
        return _case(kind, graph, v, deg, loops, fe=rng.choice([4, 8, 12, 16]))
    if kind == "sage_lstm":
        v, deg = size(500, 1 << 17, 3, 16)
        return _case(kind, graph, v, deg, loops, f_in=_logint(rng, 16, 300), hidden=rng.choice([32, 64, 128]),
                     f_out=_logint(rng, 8, 256))
    if kind == "rgcn":
        v, deg = size(1000, 1 << 18, 3, 24)
        return _case(kind, graph, v, deg, loops, dtype, f_in=_logint(rng, 16, 300), f_out=_logint(rng, 8, 128),
                     rels=_logint(rng, 2, 64), plan=rng.random() < 0.4)
    if kind == "plan":
        v, deg = size(500, 1 << 21)
        return _case(kind, graph, v, deg, loops)
    if kind == "propagate":
        v, deg = size(500, 1 << 20)
        reduce = rng.choice(["sum", "mean", "max"])
        return _case(kind, graph, v, deg, loops, dtype, reduce=reduce, norm=reduce == "sum" and rng.random() < 0.5,
                     f_in=_logint(rng, 4, 300))
    k = _logint(rng, 16, 602)
    return _case("transform", dtype=dtype, v=_logint(rng, 500, 600_000), k=k,
                 k2=k if rng.random() < 0.5 else 0, f_out=_logint(rng, 6, 300),
                 act=rng.choice(["none", "relu", "elu", "sigmoid", "tanh"]))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _tdt(case):
    return torch.bfloat16 if case["dtype"] == BF16 else torch.float32


def num_edges(case):
    """Stored edges of the case's graph (every generator makes exactly these)."""
    return case["v"] * case["deg"] + (case["v"] if case["loops"] else 0)


def _edges(case, g):
    """src, dst (int64, device) of the case's graph, before sorting."""
    v, deg = case["v"], case["deg"]
    e = v * deg

    def randint(hi, n):
        return torch.randint(hi, (n,), generator=g, device=DEV)

    if case["graph"] == "er":
        src, dst = randint(v, e), randint(v, e)
    elif case["graph"] == "rmat":
        bits = max(1, (v - 1).bit_length())
        src = torch.zeros(e, dtype=torch.int32, device=DEV)
        dst = torch.zeros(e, dtype=torch.int32, device=DEV)
        for _ in range(bits):
            q = torch.rand(e, generator=g, device=DEV)
            src.mul_(2).add_(q >= 0.76)
            dst.mul_(2).add_(((q >= 0.57) & (q < 0.76)) | (q >= 0.95))
        del q
        perm = torch.randperm(1 << bits, generator=g, device=DEV)
        src, dst = perm[src] % v, perm[dst] % v
    elif case["graph"] == "ba":
        # each new vertex sends deg/2 edges to endpoints of earlier edges
        # drawn uniformly (the linearised preferential attachment); an odd
        # draw copies the target of an earlier edge, resolved by jumping
        m = max(1, deg // 2)
        i = torch.arange(v * m, device=DEV)
        r = (torch.rand(v * m, generator=g, device=DEV, dtype=torch.float64) * (2 * i + 1)).long()
        jump = torch.where(r % 2 == 1, r // 2, i)   # edge whose target is copied (i: none)
        own = torch.where(r % 2 == 1, torch.zeros_like(r), (r // 2) // m)
        while True:
            nxt = jump[jump]
            if torch.equal(nxt, jump):
                break
            jump = nxt
        a, b = i // m, own[jump]
        src, dst = torch.cat([a, b]), torch.cat([b, a])
        src, dst = src[:e], dst[:e]
        if src.numel() < e:  # deg 1
            src, dst = randint(v, e), randint(v, e)
    else:  # mesh: near neighbours on a square torus grid, random vertex order
        side = max(2, int(math.isqrt(v)))
        half = (e + 1) // 2
        a = randint(v, half)
        reach = max(1, int(round(math.sqrt(deg))))
        off = (randint(2 * reach + 1, half) - reach) * side + randint(2 * reach + 1, half) - reach
        b = (a + off) % v
        label = torch.randperm(v, generator=g, device=DEV)
        a, b = label[a], label[b]
        src, dst = torch.cat([a, b])[:e], torch.cat([b, a])[:e]
    if case["loops"]:
        x = torch.arange(v, device=DEV)
        src, dst = torch.cat([src, x]), torch.cat([dst, x])
    return src, dst


def _csr(case, g):
    """row_ptr, col_idx (int32): rows by destination, sources ascending."""
    v = case["v"]
    src, dst = _edges(case, g)
    bits = max(1, (v - 1).bit_length())
    key = torch.sort(dst.mul_(1 << bits).add_(src)).values
    del src, dst
    col = (key & ((1 << bits) - 1)).int()
    row_ptr = torch.zeros(v + 1, dtype=torch.int32, device=DEV)
    row_ptr[1:] = torch.cumsum(torch.bincount(key >> bits, minlength=v), 0)
    return row_ptr, col


def _matrix(rows, cols, dtype, g, sparse=False):
    """rows x cols features, N(0, 1) or 5 % ones, rows padded to 16 bytes
    (the padding is NaN: it is nobody's data)."""
    per = 16 // (2 if dtype == torch.bfloat16 else 4)
    ld = (cols + per - 1) // per * per
    buf = torch.empty(rows, ld, device=DEV)
    if sparse:
        buf.uniform_(generator=g)
        buf = (buf < 0.05).to(torch.float32)
    else:
        buf.normal_(generator=g)
    if ld > cols:
        buf[:, cols:] = float("nan")
    return buf.to(dtype)[:, :cols]


def _glorot(shape, fan_in, fan_out, g, dtype=torch.float32):
    a = math.sqrt(6.0 / (fan_in + fan_out))
    return torch.empty(shape, device=DEV).uniform_(-a, a, generator=g).to(dtype)


def _bias(fan_in, n, g):
    a = 1.0 / math.sqrt(fan_in)
    return torch.empty(n, device=DEV).uniform_(-a, a, generator=g)


def _inputs(case, seed):
    """Everything the case's inputs are made of, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 12345)
    kind, v, dt = case["kind"], case["v"], _tdt(case)
    d = {}
    if kind != "transform":
        d["row_ptr"], d["col_idx"] = _csr(case, g)
    if kind == "gcn":
        fi, fh, fo = case["f_in"], case["hidden"], case["f_out"]
        d["X"] = _matrix(v, fi, dt, g, case["sparse"])
        d["W1"], d["b1"] = _glorot((fi, fh), fi, fh, g, dt), _bias(fi, fh, g)
        d["W2"], d["b2"] = _glorot((fh, fo), fh, fo, g, dt), _bias(fh, fo, g)
    elif kind == "gat":
        fi, h, hd = case["f_in"], case["heads"], case["head_dim"]
        f = h * hd
        d["X"] = _matrix(v, fi, dt, g)
        d.update(heads=h, head_dim=hd, neg_slope=0.2)
        d["W1"], d["b1"] = _glorot((fi, f), fi, f, g), _bias(fi, f, g)
        d["W2"], d["b2"] = _glorot((f, f), f, f, g), _bias(f, hd, g)
        for n in ("al1", "ar1", "al2", "ar2"):
            d[n] = _glorot((h, hd), hd, 1, g)
    elif kind == "sage_pool":
        fi, fo = case["f_in"], case["f_out"]
        d["X"] = _matrix(v, fi, dt, g)
        d["W_pool"], d["b_pool"] = _glorot((fi, fi), fi, fi, g), _bias(fi, fi, g)
        d["W"], d["b"] = _glorot((2 * fi, fo), 2 * fi, fo, g), _bias(2 * fi, fo, g)
    elif kind == "gated":
        f, fe = 64, case["fe"]
        d["H"] = _matrix(v, f, dt, g)
        d["E_feat"] = _matrix(num_edges(case), fe, dt, g)
        d["W_e"], d["b_e"] = _glorot((2 * f + fe, f), 2 * f + fe, f, g), _bias(2 * f + fe, f, g)
        for n in ("ih", "hh"):
            d["W_" + n], d["b_" + n] = _glorot((f, 3 * f), f, 3 * f, g), _bias(f, 3 * f, g)
    elif kind == "sage_lstm":
        fi, h, fo = case["f_in"], case["hidden"], case["f_out"]
        d["X"] = _matrix(v, fi, dt, g)
        a = 1.0 / math.sqrt(h)
        for n, shape in (("W_ih", (fi, 4 * h)), ("W_hh", (h, 4 * h)), ("b_ih", (4 * h,)), ("b_hh", (4 * h,))):
            d[n] = torch.empty(shape, device=DEV).uniform_(-a, a, generator=g)
        d["W"], d["b"] = _glorot((fi + h, fo), fi + h, fo, g), _bias(fi + h, fo, g)
    elif kind == "rgcn":
        fi, fo, r = case["f_in"], case["f_out"], case["rels"]
        d["X"] = _matrix(v, fi, dt, g)
        p = 1.0 / torch.arange(1, r + 1, device=DEV, dtype=torch.float64)
        edge = torch.cumsum(p / p.sum(), 0)
        u = torch.rand(num_edges(case), generator=g, device=DEV, dtype=torch.float64)
        d["etype"] = torch.bucketize(u, edge).clamp_(max=r - 1).int()
        d["W_rel"] = _glorot((r, fi, fo), fi, fo, g, dt)
        d["W_self"], d["b"] = _glorot((fi, fo), fi, fo, g, dt), _bias(fi, fo, g)
        d["act"] = "relu"
    elif kind == "propagate":
        d["X"] = _matrix(v, case["f_in"], dt, g)
    elif kind == "transform":
        k, k2, n = case["k"], case["k2"], case["f_out"]
        d["A"] = _matrix(v, k, dt, g)
        d["W"], d["b"] = _glorot((k, n), k + k2, n, g, dt), _bias(k, n, g)
        if k2:
            d["A2"] = _matrix(v, k2, dt, g)
            d["W2"] = _glorot((k2, n), k + k2, n, g, dt)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind, dt = case["kind"], _tdt(case)
    st = {"case": case, "in": d}
    if kind == "transform":
        n = case["f_out"]
        op = S.saga_gemm_op()
        op.dtype, op.act = S.dtype_code(dt), S.ACT[case["act"]]
        op.mode = S.SAGA_GEMM_CONCAT if case["k2"] else S.SAGA_GEMM_PLAIN
        st["op"] = op
        st["out"] = S.padded_empty(case["v"], n, dt, DEV)
        st["ws"] = S.workspace(S.saga_apply_vertex_workspace_size(op, case["k"], case["k2"], n), DEV)
        return st
    if kind == "plan" or case.get("plan") and kind == "rgcn":
        return st
    graph = st["graph"] = S.Graph(d["row_ptr"], d["col_idx"])
    if kind == "gcn":
        st["layers"] = LY.gcn2(graph, d["W1"], d["b1"], d["W2"], d["b2"], dtype=dt)
    elif kind == "gat":
        st["layers"] = LY.gat2(graph, d)
    elif kind == "sage_pool":
        st["layers"] = LY.sage_pool(graph, d)
    elif kind == "gated":
        st["layers"] = LY.gated_gru(graph, d)
    elif kind == "sage_lstm":
        st["layers"] = LY.sage_lstm(graph, d)
    elif kind == "rgcn":
        rel = S.RelGraph(graph, d["etype"], case["rels"])
        st["layers"] = LY.rgcn(graph, rel, d, dtype=dt)
    else:  # propagate
        op = S.saga_edge_op()
        op.msg = S.SAGA_MSG_SRC_NORM if case["norm"] else S.SAGA_MSG_COPY
        op.reduce = {"sum": S.SAGA_RED_SUM, "mean": S.SAGA_RED_MEAN, "max": S.SAGA_RED_MAX}[case["reduce"]]
        op.dtype, op.dst_norm, op.act = S.dtype_code(dt), int(case["norm"]), S.ACT["none"]
        st["op"] = op
        st["out"] = S.padded_empty(case["v"], case["f_in"], dt, DEV)
        st["ws"] = S.workspace(S.saga_gather_workspace_size(graph.plan, op, case["f_in"]), DEV)
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(st):
    case, d = st["case"], st["in"]
    kind = case["kind"]
    if kind == "plan":
        return S.Graph(d["row_ptr"], d["col_idx"]).arrays()
    if kind == "transform":
        S.saga_apply_vertex(st["op"], S.cmat(d["A"]), S.cmat(d["W"]), S.cmat(d.get("A2")), S.cmat(d.get("W2")),
                            S._ptr(d["b"]), None, S.mat(st["out"]), S._ptr(st["ws"]), st["ws"].numel(),
                            S.stream_handle())
        return st["out"]
    if kind == "propagate":
        inp = S.saga_edge_inputs()
        inp.src = S.cmat(d["X"])
        S.saga_scatter_apply_edge_gather(st["graph"].plan, st["op"], inp, S.mat(st["out"]), S._ptr(st["ws"]),
                                         st["ws"].numel(), S.stream_handle())
        return st["out"]
    if kind == "rgcn" and case["plan"]:
        graph = S.Graph(d["row_ptr"], d["col_idx"])
        rel = S.RelGraph(graph, d["etype"], case["rels"])
        return LY.run(LY.rgcn(graph, rel, d, dtype=_tdt(case)), d["X"])
    if kind == "gated":
        return LY.run(st["layers"], d["H"], edge_feat=d["E_feat"])
    if case.get("plan"):
        st["graph"].build()
    return LY.run(st["layers"], d["X"])


# --------------------------------------------------------------------------
# bytes and operations of one pass
# --------------------------------------------------------------------------
def work(case):
    kind, v = case["kind"], case["v"]
    es = 2 if case["dtype"] == BF16 else 4
    if kind == "transform":
        k, n = case["k"] + case["k2"], case["f_out"]
        return {"bytes": es * (v * k + k * n + v * n) + 4 * n, "flops": 2 * v * k * n}
    e = num_edges(case)
    csr = 4 * (e + v + 1)
    if kind == "plan":
        # the arrays handed out: degrees, order, row_seg_first; segments (at least one a row)
        return {"bytes": csr + 4 * (4 * v + 1) + 12 * v, "flops": e + v}
    if kind == "propagate":
        f = case["f_in"]
        return {"bytes": csr + 2 * es * v * f, "flops": e * f * (2 if case["norm"] else 1)}
    if kind == "gcn":
        fi, fh, fo = case["f_in"], case["hidden"], case["f_out"]
        fl = 2 * v * (fi * fh + fh * fo) + e * (min(fi, fh) + min(fh, fo))
        return {"bytes": csr + es * (v * fi + fi * fh + fh * fo + v * fo) + 4 * (fh + fo), "flops": fl}
    if kind == "gat":
        fi, h, hd = case["f_in"], case["heads"], case["head_dim"]
        f = h * hd
        fl = 2 * v * f * (fi + f) + 8 * v * f + 2 * e * (2 * f + 4 * h)
        return {"bytes": csr + 4 * (v * fi + fi * f + f * f + v * hd), "flops": fl}
    if kind == "sage_pool":
        fi, fo = case["f_in"], case["f_out"]
        return {"bytes": csr + 4 * (v * fi + fi * fi + 2 * fi * fo + v * fo),
                "flops": 2 * v * fi * (fi + 2 * fo) + e * fi}
    if kind == "gated":
        f, fe = 64, case["fe"]
        return {"bytes": csr + 4 * (2 * v * f + e * fe + (2 * f + fe) * f + 6 * f * f),
                "flops": 2 * v * f * (2 * f + 6 * f) + e * f * (2 * fe + 6)}
    if kind == "sage_lstm":
        fi, h, fo = case["f_in"], case["hidden"], case["f_out"]
        return {"bytes": csr + 4 * (v * fi + (fi + h) * 4 * h + (fi + h) * fo + v * fo),
                "flops": 2 * v * (fi * 4 * h + (fi + h) * fo) + e * (8 * h * h + 20 * h)}
    fi, fo, r = case["f_in"], case["f_out"], case["rels"]
    # at least one product per vertex and the self term; a message add per edge
    return {"bytes": csr + 4 * e + es * (v * fi + (r + 1) * fi * fo + v * fo),
            "flops": 4 * v * fi * fo + 2 * e * fo}


def tolerance(case):
    """About four times what this library shows against float64 over the
    ranges of draw(): float32 sums of up to some thousand terms in any order;
    bfloat16 with its intermediates stored in bfloat16."""
    kind = case["kind"]
    if kind == "plan":
        return "exact"
    if kind == "propagate" and case["reduce"] == "max" and not case["norm"]:
        return "exact"
    if case["dtype"] == BF16:
        return {"rel": 1e-2, "max": 5e-2}
    return {"rel": 4e-6, "max": 1e-4}


# --------------------------------------------------------------------------
# the same in float64 with plain torch
# --------------------------------------------------------------------------
def _chunks(row_ptr, rows_per):
    for lo in range(0, row_ptr.numel() - 1, rows_per):
        yield lo, min(row_ptr.numel() - 1, lo + rows_per)


def _dst(row_ptr):
    deg = (row_ptr[1:] - row_ptr[:-1]).long()
    return torch.repeat_interleave(torch.arange(deg.numel(), device=DEV), deg)


def _spmm(row_ptr, col, z, weight=None):
    """sum over in-edges of weight_e z[col_e], float64, in edge chunks."""
    v, f = row_ptr.numel() - 1, z.shape[1]
    out = torch.zeros(v, f, dtype=torch.float64, device=DEV)
    dst = _dst(row_ptr)
    step = max(1, (1 << 28) // max(1, f))
    for lo in range(0, col.numel(), step):
        m = z[col[lo:lo + step].long()]
        if weight is not None:
            m = m * weight[lo:lo + step, None]
        out.index_add_(0, dst[lo:lo + step], m)
    return out


def _spmax(row_ptr, col, z):
    v, f = row_ptr.numel() - 1, z.shape[1]
    out = torch.full((v, f), -math.inf, dtype=z.dtype, device=DEV)
    dst = _dst(row_ptr)
    step = max(1, (1 << 27) // max(1, f))
    for lo in range(0, col.numel(), step):
        i = dst[lo:lo + step, None].expand(-1, f)
        out.scatter_reduce_(0, i, z[col[lo:lo + step].long()], "amax")
    return torch.where(torch.isinf(out), torch.zeros_like(out), out)


def _mm(x, w):
    """x w in float64, x widened in row chunks."""
    w = w.double()
    out = torch.empty(x.shape[0], w.shape[1], dtype=torch.float64, device=DEV)
    step = 1 << 18
    for lo in range(0, x.shape[0], step):
        out[lo:lo + step] = x[lo:lo + step].double() @ w
    return out


def _inv_sqrt(deg):
    d = deg.double()
    return torch.where(d > 0, d.clamp(min=1).rsqrt(), torch.zeros_like(d))


def _act(name, x):
    return {"none": lambda t: t, "relu": torch.relu, "sigmoid": torch.sigmoid, "tanh": torch.tanh,
            "elu": torch.nn.functional.elu}[name](x)


def _exact_plan(d):
    """The arrays of include/saga.h's plan section with the default options."""
    rp, col = d["row_ptr"].long(), d["col_idx"].long()
    v, e = rp.numel() - 1, col.numel()
    din = rp[1:] - rp[:-1]
    b = 256
    while b < 4096 and b * 2 <= (e + 4 * v) // 2048:
        b *= 2
    t = min(b // 2, 512)
    while b < t + 4:
        b *= 2
    perm = torch.sort(-din, stable=True).indices
    dp = din[perm]
    nseg = torch.where(dp > t, (dp + t - 1) // t, torch.ones_like(dp))
    first = torch.zeros(v + 1, dtype=torch.int64, device=DEV)
    first[1:] = torch.cumsum(nseg, 0)
    pos = torch.repeat_interleave(torch.arange(v, device=DEV), nseg)
    j = torch.arange(pos.numel(), device=DEV) - first[pos]
    row = perm[pos]
    beg = rp[row] + j * t
    end = torch.where(dp[pos] > t, torch.minimum(beg + t, rp[row + 1]), rp[row + 1])
    cost = end - beg + 4
    blk = (torch.cumsum(cost, 0) - cost) // b
    nb = int(blk[-1]) + 1
    ptr = torch.searchsorted(blk, torch.arange(nb + 1, device=DEV))
    out = dict(d_in=din, d_out=torch.bincount(col, minlength=v), perm=perm, row_seg_first=first, seg_row=row,
               seg_beg=beg, seg_end=end, block_ptr=ptr)
    return {k: x.int() for k, x in out.items()}


def _exact_lstm(d, p):
    """Last hidden state of the LSTM over each row's in-edges; p: the input half of the gates."""
    rp, col = d["row_ptr"].long(), d["col_idx"].long()
    deg = rp[1:] - rp[:-1]
    order = torch.sort(-deg, stable=True).indices
    whh = d["W_hh"].double()
    h_dim = whh.shape[0]
    v = deg.numel()
    h = torch.zeros(v, h_dim, dtype=torch.float64, device=DEV)
    c = torch.zeros_like(h)
    beg = rp[:-1][order]
    counts = torch.bincount(deg).cpu()
    active = v - torch.cumsum(counts, 0)  # active[t]: rows longer than t
    for t in range(counts.numel() - 1):
        n = int(active[t])
        z = p[col[beg[:n] + t]] + h[:n] @ whh
        i, f, o = (torch.sigmoid(z[:, k * h_dim:(k + 1) * h_dim]) for k in (0, 1, 3))
        cn = f * c[:n] + i * torch.tanh(z[:, 2 * h_dim:3 * h_dim])
        c[:n] = cn
        h[:n] = o * torch.tanh(cn)
    out = torch.empty_like(h)
    out[order] = h
    return out


def _exact_gat(d, x, w, al, ar, b, mean):
    h, hd = d["heads"], d["head_dim"]
    rp, col, dst = d["row_ptr"], d["col_idx"].long(), _dst(d["row_ptr"])
    v = rp.numel() - 1
    z = _mm(x, w)
    zh = z.view(v, h, hd)
    el, er = (zh * al.double()).sum(2), (zh * ar.double()).sum(2)
    s = torch.nn.functional.leaky_relu(el[col] + er[dst], d["neg_slope"])
    m = torch.full((v, h), -math.inf, dtype=torch.float64, device=DEV)
    m.scatter_reduce_(0, dst[:, None].expand(-1, h), s, "amax")
    p = torch.exp(s - m[dst])
    norm = torch.zeros(v, h, dtype=torch.float64, device=DEV).index_add_(0, dst, p)
    out = torch.zeros(v, h, hd, dtype=torch.float64, device=DEV)
    for k in range(h):
        out[:, k] = _spmm(rp, d["col_idx"], zh[:, k].contiguous(), p[:, k])
    out /= norm.clamp(min=1e-300)[:, :, None]
    if mean:
        return out.mean(1) + b.double()
    return torch.nn.functional.elu(out.reshape(v, h * hd) + b.double())


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "plan":
        return _exact_plan(d)
    if kind == "transform":
        z = _mm(d["A"], d["W"])
        if case["k2"]:
            z += _mm(d["A2"], d["W2"])
        return _act(case["act"], z + d["b"].double())
    rp, col = d["row_ptr"], d["col_idx"]
    din = (rp[1:] - rp[:-1]).long()
    if kind == "propagate":
        if case["reduce"] == "max":
            return _spmax(rp, col, d["X"].double())
        dout = torch.bincount(col.long(), minlength=case["v"])
        x = d["X"].double()
        if case["norm"]:
            return _spmm(rp, col, x * _inv_sqrt(dout)[:, None]) * _inv_sqrt(din)[:, None]
        s = _spmm(rp, col, x)
        return s / din.clamp(min=1)[:, None] if case["reduce"] == "mean" else s
    if kind == "gcn":
        dout = torch.bincount(col.long(), minlength=case["v"])
        h = None
        for w, b, act in ((d["W1"], d["b1"], "relu"), (d["W2"], d["b2"], "none")):
            z = _mm(d["X"] if h is None else h, w)
            z *= _inv_sqrt(dout)[:, None]
            h = _act(act, _spmm(rp, col, z) * _inv_sqrt(din)[:, None] + b.double())
        return h
    if kind == "gat":
        h = _exact_gat(d, d["X"], d["W1"], d["al1"], d["ar1"], d["b1"], False)
        return _exact_gat(d, h, d["W2"], d["al2"], d["ar2"], d["b2"], True)
    if kind == "sage_pool":
        f = case["f_in"]
        a = _spmax(rp, col, torch.relu(_mm(d["X"], d["W_pool"]) + d["b_pool"].double()))
        return _mm(d["X"], d["W"][:f]) + _mm(a, d["W"][f:]) + d["b"].double()
    if kind == "sage_lstm":
        f = case["f_in"]
        a = _exact_lstm(d, _mm(d["X"], d["W_ih"]) + (d["b_ih"].double() + d["b_hh"].double()))
        return _mm(d["X"], d["W"][:f]) + _mm(a, d["W"][f:]) + d["b"].double()
    if kind == "gated":
        f = 64
        h, dst = d["H"].double(), _dst(rp)
        we = d["W_e"].double()
        gs, gd = h @ we[:f], h @ we[f:2 * f]
        a = torch.zeros_like(h)
        step = 1 << 21
        for lo in range(0, col.numel(), step):
            u, t = col[lo:lo + step].long(), dst[lo:lo + step]
            gate = torch.sigmoid(gs[u] + gd[t] + d["b_e"].double() + d["E_feat"][lo:lo + step].double() @ we[2 * f:])
            a.index_add_(0, t, gate * h[u])
        gi = a @ d["W_ih"].double() + d["b_ih"].double()
        gh = h @ d["W_hh"].double() + d["b_hh"].double()
        r, z = torch.sigmoid(gi[:, :f] + gh[:, :f]), torch.sigmoid(gi[:, f:2 * f] + gh[:, f:2 * f])
        n = torch.tanh(gi[:, 2 * f:] + r * gh[:, 2 * f:])
        return (1 - z) * n + z * h
    # rgcn
    v, r = case["v"], case["rels"]
    et, dst = d["etype"].long(), _dst(rp)
    cnt = torch.bincount(dst * r + et, minlength=v * r)
    norm = 1.0 / cnt[dst * r + et].double()
    out = _mm(d["X"], d["W_self"]) + d["b"].double()
    for k in range(r):
        e = torch.nonzero(et == k).flatten()
        if e.numel():
            out.index_add_(0, dst[e], _mm(d["X"], d["W_rel"][k])[col[e].long()] * norm[e, None])
    return torch.relu(out)
