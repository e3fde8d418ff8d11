"""float32 products on the bfloat16 matrix cores (three-way split of both
operands): edges of the column tiles, k chunks and row tiles, both operands of
the concat form, and values outside the split's range, which take the float32
instruction.  Reference: float64 on the CPU.

Bound: six exact partial products of a w, the neglected ones together below
2^-24 |a w|, accumulated in float32 (an error of at most (K + 6) 2^-24 sum |a w|)."""
import numpy as np
import pytest
import torch

from paper_2009_00804_amd import saga as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _mat(x):
    """device matrix with 16-byte rows, the padding NaN"""
    ld = (x.shape[1] + 3) // 4 * 4
    buf = torch.full((x.shape[0], ld), float("nan"), device=DEV)
    buf[:, :x.shape[1]] = torch.from_numpy(x)
    return buf[:, :x.shape[1]]


def _run(a, w, a2=None, w2=None, bias=None):
    op = S.saga_gemm_op()
    op.mode = S.SAGA_GEMM_PLAIN if a2 is None else S.SAGA_GEMM_CONCAT
    M, K = a.shape
    N, K2 = w.shape[1], 0 if a2 is None else a2.shape[1]
    out = S.padded_empty(M, N, torch.float32, DEV)
    out.fill_(float("nan"))
    ws = S.workspace(S.saga_apply_vertex_workspace_size(op, K, K2, N), DEV)
    t = [None if x is None else torch.from_numpy(x).to(DEV) for x in (w, w2, bias)]
    am, am2 = _mat(a), None if a2 is None else _mat(a2)
    S.saga_apply_vertex(op, S.cmat(am), S.cmat(t[0]), S.cmat(am2), S.cmat(t[1]), S._ptr(t[2]), None,
                        S.mat(out), S._ptr(ws), ws.numel(), S.stream_handle())
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _check(got, a, w, a2=None, w2=None, bias=None):
    ref = a.astype(np.float64) @ w
    mag = np.abs(a).astype(np.float64) @ np.abs(w)
    K = a.shape[1]
    if a2 is not None:
        ref += a2.astype(np.float64) @ w2
        mag += np.abs(a2).astype(np.float64) @ np.abs(w2)
        K += a2.shape[1]
    if bias is not None:
        ref, mag = ref + bias, mag + np.abs(bias)
    assert np.all(np.abs(got - ref) <= (K + 6) * 2.0 ** -24 * mag + 1e-38)


@pytest.mark.parametrize("M,K,N", [
    (1, 1, 33), (15, 31, 41), (64, 32, 48), (65, 33, 64), (63, 64, 80), (129, 65, 96), (127, 96, 112),
    (130, 97, 128), (200, 128, 129), (77, 160, 200), (300, 602, 128), (128, 289, 16), (50, 300, 7),
    (33, 64, 1000), (131072 + 5, 256, 40), (70001, 259, 257)])
def test_plain(M, K, N):
    rng = np.random.default_rng(M * 7 + K * 3 + N)
    a = rng.standard_normal((M, K), dtype=np.float32)
    w = rng.uniform(-1, 1, (K, N)).astype(np.float32)
    b = rng.uniform(-1, 1, N).astype(np.float32)
    _check(_run(a, w, bias=b), a, w, bias=b)


@pytest.mark.parametrize("M,K,K2,N", [(1, 32, 1, 40), (129, 1, 33, 130), (100, 100, 64, 64), (90, 64, 256, 200),
                                      (131072, 130, 127, 136)])
def test_concat(M, K, K2, N):
    rng = np.random.default_rng(M + K + K2 + N)
    a, a2 = (rng.standard_normal((M, k), dtype=np.float32) for k in (K, K2))
    w, w2 = (rng.uniform(-1, 1, (k, N)).astype(np.float32) for k in (K, K2))
    _check(_run(a, w, a2, w2), a, w, a2, w2)


@pytest.mark.parametrize("M,K,N", [(150, 70, 50), (40, 300, 130)])
def test_values_outside_the_split(M, K, N):
    """Huge, tiny and non-finite rows and columns among ordinary ones."""
    rng = np.random.default_rng(K)
    a = rng.standard_normal((M, K), dtype=np.float32)
    w = rng.uniform(-1, 1, (K, N)).astype(np.float32)
    a[3] *= np.float32(1e30)
    a[20] *= np.float32(1e-36)
    a[21] = 0
    w[:, 5] *= np.float32(1e-37)
    _check(_run(a, w), a, w)
    w[:, 6] *= np.float32(1e25)
    w[2, 7] = np.float32(3.4e38)
    a[3], a[20] = 1, 2
    a[:, 2] = np.float32(0.5)  # the products stay finite
    _check(_run(a, w), a, w)


def test_infinities_and_nan():
    rng = np.random.default_rng(5)
    a = rng.standard_normal((100, 64), dtype=np.float32)
    w = rng.uniform(0.5, 1, (64, 40)).astype(np.float32)
    a[7, 3], a[8, 4], a[9, 5] = np.inf, -np.inf, np.nan
    a[10, 1], a[10, 2] = np.inf, -np.inf
    w[:, 1] = 1  # exactly one bfloat16: its split has zero parts
    w[6, 2] = np.inf
    got = _run(a, w)
    with np.errstate(invalid="ignore"):
        ref = a.astype(np.float64) @ w
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf])
    fin = np.isfinite(ref)
    assert np.allclose(got[fin], ref[fin], rtol=1e-5, atol=1e-4)


def _sig(x):
    return 1 / (1 + np.exp(-x))


def _gru(a, h, w, w2, b, b2):
    F = h.shape[1]
    with np.errstate(over="ignore"):
        gi, gh = a @ w + b, h @ w2 + b2
        r, z = _sig(gi[:, :F] + gh[:, :F]), _sig(gi[:, F:2 * F] + gh[:, F:2 * F])
        n = np.tanh(gi[:, 2 * F:] + r * gh[:, 2 * F:])
    return (1 - z) * n + z * h


def _run_gru(a, h, w, w2, b, b2):
    (M, K), F = a.shape, h.shape[1]
    op = S.saga_gemm_op()
    op.mode = S.SAGA_GEMM_GRU
    t = [torch.from_numpy(x).to(DEV) for x in (w, w2, b, b2)]
    am, hm = _mat(a), _mat(h)
    out = S.padded_empty(M, F, torch.float32, DEV)
    ws = S.workspace(S.saga_apply_vertex_workspace_size(op, K, F, 3 * F), DEV)
    S.saga_apply_vertex(op, S.cmat(am), S.cmat(t[0]), S.cmat(hm), S.cmat(t[1]), S._ptr(t[2]), S._ptr(t[3]),
                        S.mat(out), S._ptr(ws), ws.numel(), S.stream_handle())
    return out.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("M,K,F,special", [(1, 1, 16, False), (65, 33, 32, False), (130, 70, 48, False),
                                           (200, 64, 64, False), (64, 5, 64, True)])
def test_gru(M, K, F, special):
    """Both products share the r and z accumulators; the gates' slopes are at most
    1, so the products' bound carries over to the new state."""
    rng = np.random.default_rng(M + K + F)
    a = rng.standard_normal((M, K), dtype=np.float32)
    h = rng.standard_normal((M, F), dtype=np.float32)
    w, w2 = (rng.uniform(-0.3, 0.3, (k, 3 * F)).astype(np.float32) for k in (K, F))
    b, b2 = (rng.uniform(-1, 1, 3 * F).astype(np.float32) for _ in range(2))
    if special:  # a row past the split's range: its gates saturate
        a[5] *= np.float32(1e30)
    ref = _gru(*(x.astype(np.float64) for x in (a, h, w, w2, b, b2)))
    assert np.abs(_run_gru(a, h, w, w2, b, b2) - ref).max() <= 2e-5


@pytest.mark.parametrize("Fi,heads,D,mean", [(3, 1, 4, False), (33, 2, 4, True), (100, 8, 16, False), (64, 8, 8, True)])
def test_attention_vectors_folded_into_the_weights(Fi, heads, D, mean):
    """GAT layer against the oracle: z, el and er come from one product."""
    from gpu_util import dev_padded, graph
    from synth import graphs as G

    V = 300
    rng = np.random.default_rng(Fi)
    src, dst = rng.integers(0, V, 1500), rng.integers(0, V, 1500)
    rp, col = G.to_in_csr(V, src, dst)
    F = heads * D
    x = rng.standard_normal((V, Fi), dtype=np.float32)
    w = rng.uniform(-0.5, 0.5, (Fi, F)).astype(np.float32)
    al, ar = (rng.uniform(-1, 1, (heads, D)).astype(np.float32) for _ in range(2))
    b = rng.uniform(-1, 1, D if mean else F).astype(np.float32)
    from paper_2009_00804_amd import layers as LY
    g = graph(rp, col)
    layer = LY.Layer(g, "gat", Fi, D if mean else F, {"w": w, "b": b, "attn_l": al, "attn_r": ar}, heads=heads,
                     head_mean=mean, act="none")
    got = layer(dev_padded(x)).cpu().numpy().astype(np.float64)
    z = (x.astype(np.float64) @ w).reshape(V, heads, D)
    el, er = (z * al).sum(2), (z * ar).sum(2)
    ref = np.zeros((V, heads, D))
    for v in range(V):
        u = col[rp[v]:rp[v + 1]]
        if u.size:
            s = el[u] + er[v]
            s = np.where(s > 0, s, 0.2 * s)
            p = np.exp(s - s.max(0))
            ref[v] = (p[:, :, None] * z[u]).sum(0) / p.sum(0)[:, None]
    ref = (ref.mean(1) if mean else ref.reshape(V, F)) + b
    assert np.abs(got - ref).max() <= 1e-4 * max(1.0, np.sqrt((ref ** 2).mean()))
