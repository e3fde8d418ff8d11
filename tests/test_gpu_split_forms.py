"""The float32 split path in every form it takes: attention vectors folded into
tiles with few or many folded columns, long grouped products, and values outside
the split's range (m w K of 2^94 and more, or infinite), which take the float32
instruction, in each operand of each form.  Reference: float64 on the CPU."""
import numpy as np
import pytest
import torch

import test_gpu_rgcn as R
from gpu_util import dev_padded, graph
from oracle import saga_oracle as O
from paper_2009_00804_amd import layers as LY
from synth import graphs as G
from test_gpu_split_gemm import _check, _gru, _run
from test_gpu_split_gemm import test_attention_vectors_folded_into_the_weights as check_folded

pytestmark = pytest.mark.gpu


# folded columns of a tile: 2 (one head), 4 + 2, 4, 10, 12, 4 + 10, 6
@pytest.mark.parametrize("Fi,heads,D,mean", [(5, 1, 64, False), (130, 1, 16, True), (7, 3, 4, False), (40, 2, 32, False),
                                             (9, 5, 4, False), (129, 6, 8, False), (33, 7, 4, False), (20, 3, 8, False)])
def test_folded_columns_of_a_tile(Fi, heads, D, mean):
    check_folded(Fi, heads, D, mean)


def _normal(rng, *shape):
    return rng.standard_normal(shape, dtype=np.float32)


@pytest.mark.parametrize("operand", [0, 1])
@pytest.mark.parametrize("M,K,K2,N", [(70, 40, 33, 150), (131072, 200, 64, 136)])
def test_concat_values_outside_the_split(operand, M, K, K2, N):
    """A huge column, a huge and an infinite row in either operand."""
    rng = np.random.default_rng(K + operand)
    a, w = [_normal(rng, M, K), _normal(rng, M, K2)], [_normal(rng, K, N), _normal(rng, K2, N)]
    rows = np.unique(np.concatenate([np.arange(64), rng.integers(0, M, 500), [M - 1]]))
    w[operand][:, 17] *= np.float32(2.0 ** 98)
    print(f"concat {operand} {M}", flush=True)
    got = _run(a[0], w[0], a[1], w[1])
    _check(got[rows], a[0][rows], w[0], a[1][rows], w[1])
    w[operand][:, 17] = 1
    a[operand][5] *= np.float32(2.0 ** 100)
    a[operand][40, 3], w[operand][3, :] = np.inf, 0.5
    got = _run(a[0], w[0], a[1], w[1])
    assert np.all(got[40] == np.inf)
    rows = rows[rows != 40]
    _check(got[rows], a[0][rows], w[0], a[1][rows], w[1])


@pytest.mark.parametrize("K,N", [(225, 40), (300, 128), (257, 200), (602, 16)])
def test_long_grouped_products(K, N):
    """Eight and more k chunks: 32 rows a wave."""
    for case in (R.CASES[4], R.CASES[6]):
        _grouped(case, K, N, lambda X, W: None)


@pytest.mark.parametrize("K,N", [(40, 50), (230, 150)])
@pytest.mark.parametrize("what", ["column", "row"])
def test_grouped_values_outside_the_split(K, N, what):
    def change(X, W):
        if what == "column":
            W[2, :, N - 3] *= np.float32(2.0 ** 97)
        else:
            X[::7] *= np.float32(2.0 ** 97)

    _grouped(R.CASES[4], K, N, change)


def _grouped(case, K, N, change):
    name, n, nrel, rp, col, et = case
    print(f"grouped {name} {K} x {N}", flush=True)
    _, rg = R._rel(n, nrel, rp, col, et)
    rng = np.random.default_rng(K * N)
    X, W = _normal(rng, n, K), _normal(rng, nrel, K, N)
    change(X, W)
    got = R._run_transform(rg, X, W, "f32")
    L = O.rel_layout(rp, col, et, nrel, R.TILE)
    for r in range(nrel):
        q = slice(L["rel_ptr"][r], L["rel_ptr"][r] + L["rel_count"][r])
        _check(got[q], X[L["pair_src"][q]], W[r])


def _small_graph(rng, V, E):
    return G.to_in_csr(V, rng.integers(0, V, E), rng.integers(0, V, E))


@pytest.mark.parametrize("vector", ["w", "al", "ar"])
def test_folded_values_outside_the_split(vector):
    """A huge attention vector: scores of 2^100, so that the softmax takes the
    largest alone; a huge weight column nobody's score uses."""
    V, Fi, heads, D = 150, 40, 4, 8
    rng = np.random.default_rng(len(vector))
    rp, col = _small_graph(rng, V, 900)
    x, w = _normal(rng, V, Fi), _normal(rng, Fi, heads * D)
    a = {k: _normal(rng, heads, D) for k in ("al", "ar")}
    if vector == "w":
        w[:, 11] *= np.float32(2.0 ** 95)
        a["al"][1, 3] = a["ar"][1, 3] = 0
    else:
        a[vector] *= np.float32(2.0 ** 96)
    layer = LY.Layer(graph(rp, col), "gat", Fi, heads * D,
                     {"w": w, "b": np.zeros(heads * D, np.float32), "attn_l": a["al"], "attn_r": a["ar"]},
                     heads=heads, act="none")
    got = layer(dev_padded(x)).cpu().numpy().astype(np.float64).reshape(V, heads, D)
    z = (x.astype(np.float64) @ w).reshape(V, heads, D)
    el, er = (z * a["al"]).sum(2), (z * a["ar"]).sum(2)
    scale = np.abs(z).max((0, 1))  # per column: the huge one does not hide the others
    for v in range(V):
        u = col[rp[v]:rp[v + 1]]
        if u.size:
            s = el[u] + er[v]
            s = np.where(s > 0, s, 0.2 * s)
            p = np.exp(s - s.max(0))
            ref = (p[:, :, None] * z[u]).sum(0) / p.sum(0)[:, None]
            assert np.all(np.abs(got[v] - ref) <= 1e-4 * scale), v


@pytest.mark.parametrize("block", [0, 1])
def test_gate_blocks_outside_the_split(block):
    """A huge column in either block of W_e: its gate is 0 or 1."""
    V, F, Fe = 200, 64, 8
    rng = np.random.default_rng(block)
    rp, col = _small_graph(rng, V, 1500)
    h, ef = _normal(rng, V, F), _normal(rng, col.size, Fe)
    w = {"w_e": 0.2 * _normal(rng, 2 * F + Fe, F), "b_e": _normal(rng, F), "w_ih": 0.1 * _normal(rng, F, 3 * F),
         "b_ih": _normal(rng, 3 * F), "w_hh": 0.1 * _normal(rng, F, 3 * F), "b_hh": _normal(rng, 3 * F)}
    w["w_e"][block * F:(block + 1) * F, 21] *= np.float32(2.0 ** 100)
    layer = LY.Layer(graph(rp, col), "gated_gru", F, F, w, edge_feat=Fe)
    got = layer(dev_padded(h), edge_feat=dev_padded(ef)).cpu().numpy().astype(np.float64)
    w = {k: x.astype(np.float64) for k, x in w.items()}
    h = h.astype(np.float64)
    dst = np.repeat(np.arange(V), np.diff(rp))
    with np.errstate(over="ignore"):
        gate = 1 / (1 + np.exp(-((h @ w["w_e"][:F])[col] + (h @ w["w_e"][F:2 * F])[dst] + ef @ w["w_e"][2 * F:] + w["b_e"])))
    a = np.zeros((V, F))
    np.add.at(a, dst, gate * h[col])
    assert np.abs(got - _gru(a, h, w["w_ih"], w["w_hh"], w["b_ih"], w["b_hh"])).max() <= 1e-4


@pytest.mark.parametrize("what", ["w", "w2", "a", "h"])
@pytest.mark.parametrize("F", [16, 64])
def test_gru_values_outside_the_split(what, F):
    """Huge columns (r, z and n gates) or rows: the gates saturate."""
    from test_gpu_split_gemm import _run_gru

    M, K = 100, 40
    rng = np.random.default_rng(F)
    a, h = _normal(rng, M, K), _normal(rng, M, F)
    w, w2, b, b2 = _normal(rng, K, 3 * F), _normal(rng, F, 3 * F), _normal(rng, 3 * F), _normal(rng, 3 * F)
    if what in ("w", "w2"):
        (w if what == "w" else w2)[:, [3, F + 4, 2 * F + 5]] *= np.float32(2.0 ** 96)
    elif what == "a":
        a[::9] *= np.float32(2.0 ** 96)
    else:
        h[::9] *= np.float32(2.0 ** 96)
    got = _run_gru(a, h, w, w2, b, b2)
    ref = _gru(*(x.astype(np.float64) for x in (a, h, w, w2, b, b2)))
    scale = np.maximum(np.abs(h).max(1), 1)[:, None]  # z h carries a huge row through
    assert np.all(np.abs(got - ref) <= 2e-5 * scale)
