"""float32 products on the bfloat16 matrix cores are no further from float64
than float32 sums with one rounding per product, whatever the inputs' zeros:
dense rows, rows after ReLU, rows with few nonzeros.

Reference: float64 on the CPU.  Yardstick: the float32 sum in the order of k, a
fused multiply-add per product (emulated in float64 and rounded).  The terms the
split leaves out add 2^-27.5 |a w| in the root mean square to a single product's
2^-25.2: 2.1 % at one nonzero a row, less with more; the statistic over 30,000
outputs scatters by 0.5 %."""
import numpy as np
import pytest

from test_gpu_split_gemm import _run

pytestmark = pytest.mark.gpu
ROWS = 512


def _fma_sum(pairs):
    acc = None
    for a, w in pairs:
        a, w = a.astype(np.float64), w.astype(np.float64)
        for k in range(a.shape[1]):
            p = a[:, k, None] * w[k]
            acc = (p if acc is None else acc.astype(np.float64) + p).astype(np.float32)
    return acc.astype(np.float64)


def _rows(rng, kind, M, K):
    x = rng.standard_normal((M, K), dtype=np.float32)
    if kind == "relu":
        return np.maximum(x, 0)
    if kind.startswith("sparse"):
        x[rng.random((M, K), dtype=np.float32) >= float(kind[6:])] = 0
    if kind == "bag":  # row-normalized counts
        x = (rng.random((M, K), dtype=np.float32) < 0.05).astype(np.float32)
        x /= np.maximum(x.sum(1, keepdims=True), 1)
    return x


def _rms(got, ref):
    return np.sqrt(((got - ref) ** 2).mean())


@pytest.mark.parametrize("kind", ["dense", "relu", "sparse0.1", "sparse0.02", "sparse0.004", "bag"])
@pytest.mark.parametrize("M,K,K2,N", [(ROWS, 602, 0, 64), (ROWS, 96, 0, 130), (ROWS, 130, 70, 64),
                                      (131072, 300, 0, 128), (131072, 200, 200, 128)])
def test_no_further_from_float64_than_float32_sums(kind, M, K, K2, N):
    rng = np.random.default_rng(K + K2 + N)
    a = [_rows(rng, kind, M, k) for k in (K, K2) if k]
    w = [rng.uniform(-1, 1, (k, N)).astype(np.float32) for k in (K, K2) if k]
    print(f"{kind} {M} x {K}+{K2} x {N}", flush=True)
    got = _run(a[0], w[0], *((a[1], w[1]) if K2 else ()))
    pick = rng.permutation(M)[:ROWS]
    ref = sum(x[pick].astype(np.float64) @ y for x, y in zip(a, w))
    plain = _rms(_fma_sum([(x[pick], y) for x, y in zip(a, w)]), ref)
    assert _rms(got[pick], ref) <= 1.04 * plain


def _bound(a, w):
    """a float32 sum of the split's terms, plus one rounding of a subnormal result"""
    mag = np.abs(a).astype(np.float64) @ np.abs(w).astype(np.float64)
    return (a.shape[1] + 6) * 2.0 ** -24 * mag + 2.0 ** -149


@pytest.mark.parametrize("e", [60, 105, 112, 120, 126, 130, 140, 148])
def test_elements_far_below_their_row_and_column(e):
    """Values down to the smallest subnormal keep their bits beside ordinary ones
    (here: meet a zero), in either operand."""
    rng = np.random.default_rng(e)
    tiny = (rng.uniform(1, 2, 64) * 2.0 ** -e).astype(np.float32)
    big = (rng.uniform(1, 2, 64) * 2.0 ** 40).astype(np.float32)
    one = rng.uniform(1, 2, 64).astype(np.float32)
    zero = np.zeros(64, np.float32)
    a, w = np.stack([one, tiny], 1), np.stack([zero, big])
    assert np.all(np.abs(_run(a, w) - a.astype(np.float64) @ w) <= _bound(a, w))
    a, w = np.stack([zero, big], 1), np.stack([one, tiny])
    assert np.all(np.abs(_run(a, w) - a.astype(np.float64) @ w) <= _bound(a, w))


@pytest.mark.parametrize("ea,ew", [(-45, 0), (0, -45), (-60, -60), (-70, -64), (61, 20), (20, 61), (90, -60), (-100, 109),
                                   (70, 17), (70, 18), (71, 18), (109, -30), (111, -30), (-30, 111), (100, 20),
                                   (-140, 30)])
def test_magnitudes_around_the_split_range(ea, ew):
    """Small and large operands, on both sides of where the float32 instruction
    takes over (2^110 in either operand, 2^94 for their product and K)."""
    rng = np.random.default_rng((ea + 200) * 400 + ew + 200)
    a = np.ldexp(rng.uniform(0.5, 1, (70, 64)).astype(np.float32) * rng.choice([-1, 1], (70, 64)), ea)
    w = np.ldexp(rng.uniform(0.5, 1, (64, 48)).astype(np.float32) * rng.choice([-1, 1], (64, 48)), ew)
    a, w = a.astype(np.float32), w.astype(np.float32)
    assert np.all(np.abs(_run(a, w) - a.astype(np.float64) @ w) <= _bound(a, w) + 64 * 2.0 ** -149)


@pytest.mark.parametrize("K", [1, 2, 3, 4])
def test_few_k(K):
    """Up to four k every term counts: a product is rounded as a float32 one is."""
    rng = np.random.default_rng(K)
    a, w = rng.standard_normal((4096, K), dtype=np.float32), rng.uniform(-1, 1, (K, 64)).astype(np.float32)
    ref = a.astype(np.float64) @ w
    assert _rms(_run(a, w), ref) <= 1.005 * _rms(_fma_sum([(a, w)]), ref)
