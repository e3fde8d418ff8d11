"""bfloat16 products with more than 80 columns: edges of the column blocks (one
block up to 13 column tiles, blocks of at most ten past that, of seven over few rows), k chunks of 64, row
tiles, both operands of the concat form, the split output.

Reference: float64 of the bfloat16 inputs.  Bound: products exact in float32,
sums of K terms (K 2^-24 of the magnitudes), one rounding to bfloat16."""
import numpy as np
import pytest
import torch

from gpu_util import dev_padded, to_np
from paper_2009_00804_amd import saga as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bf(x):
    return torch.from_numpy(x).to(torch.bfloat16).to(torch.float64).numpy()


@pytest.mark.parametrize("M,K,K2,N,split", [
    (1, 1, 0, 81, 0), (63, 63, 0, 96, 0), (64, 64, 0, 112, 64), (65, 65, 0, 128, 0), (200, 128, 0, 129, 0),
    (130, 129, 0, 200, 128), (70, 191, 0, 256, 0), (33, 40, 0, 257, 0), (50, 100, 0, 300, 0),
    (131071, 24, 0, 208, 0), (131072, 72, 0, 209, 0), (65536, 449, 0, 100, 64), (40001, 33, 0, 260, 0),
    (400001, 16, 0, 88, 0), (32767, 72, 0, 200, 0), (32768, 72, 0, 200, 0), (65537, 16, 448, 90, 0),
    (100, 64, 1, 90, 0), (129, 1, 65, 144, 0), (300, 300, 300, 200, 0), (33000, 130, 40, 170, 0),
    (77, 700, 0, 128, 0), (31, 8, 8, 1000, 0)])
def test_products(M, K, K2, N, split):
    rng = np.random.default_rng(M + K + K2 + N)
    a = [rng.standard_normal((M, k), dtype=np.float32) for k in (K, K2) if k]
    w = [rng.uniform(-1, 1, (k, N)).astype(np.float32) for k in (K, K2) if k]
    b = rng.uniform(-1, 1, N).astype(np.float32)
    op = S.saga_gemm_op()
    op.dtype, op.mode = S.SAGA_BF16, S.SAGA_GEMM_CONCAT if K2 else S.SAGA_GEMM_PLAIN
    out = S.padded_empty(M, split or N, torch.bfloat16, DEV)
    tail = S.padded_empty(M, N - split, torch.bfloat16, DEV) if split else None
    if split:
        op.split_col, op.tail = split, S.mat(tail)
    ad = [dev_padded(x, torch.bfloat16) for x in a] + [None]
    wd = [torch.from_numpy(x).to(DEV).to(torch.bfloat16) for x in w] + [None]
    bd = torch.from_numpy(b).to(DEV)
    ws = S.workspace(S.saga_apply_vertex_workspace_size(op, K, K2, N), DEV)
    S.saga_apply_vertex(op, S.cmat(ad[0]), S.cmat(wd[0]), S.cmat(ad[1]), S.cmat(wd[1]), S._ptr(bd), None,
                        S.mat(out), S._ptr(ws), ws.numel(), S.stream_handle())
    got = np.concatenate([to_np(out), to_np(tail)], 1) if split else to_np(out)
    ref = sum(_bf(x) @ _bf(y) for x, y in zip(a, w)) + b
    mag = sum(np.abs(_bf(x)) @ np.abs(_bf(y)) for x, y in zip(a, w)) + np.abs(b)
    assert np.all(np.abs(got - ref) <= (K + K2 + 2) * 2.0 ** -24 * mag + 2.0 ** -8 * np.abs(ref) + 1e-30)


@pytest.mark.parametrize("M,K,K2,N", [(131072, 70, 0, 140), (131072 + 77, 65, 0, 160), (131073, 130, 66, 170),
                                      (140000, 72, 40, 190), (131072, 200, 0, 208), (150001, 129, 64, 200)])
def test_products_of_many_rows(M, K, K2, N):
    """9 to 13 column tiles over 131,072 rows and more: eight waves a workgroup.
    A thousand rows are compared, the last tile's among them."""
    rng = np.random.default_rng(M + K + K2 + N)
    a = [rng.standard_normal((M, k), dtype=np.float32) for k in (K, K2) if k]
    w = [rng.uniform(-1, 1, (k, N)).astype(np.float32) for k in (K, K2) if k]
    op = S.saga_gemm_op()
    op.dtype, op.mode = S.SAGA_BF16, S.SAGA_GEMM_CONCAT if K2 else S.SAGA_GEMM_PLAIN
    out = S.padded_empty(M, N, torch.bfloat16, DEV)
    out.fill_(float("nan"))
    ad = [dev_padded(x, torch.bfloat16) for x in a] + [None]
    wd = [torch.from_numpy(x).to(DEV).to(torch.bfloat16) for x in w] + [None]
    ws = S.workspace(S.saga_apply_vertex_workspace_size(op, K, K2, N), DEV)
    print(f"stream {M} x {K}+{K2} x {N}", flush=True)
    S.saga_apply_vertex(op, S.cmat(ad[0]), S.cmat(wd[0]), S.cmat(ad[1]), S.cmat(wd[1]), None, None, S.mat(out),
                        S._ptr(ws), ws.numel(), S.stream_handle())
    assert not bool(torch.isnan(out).any())
    rows = np.unique(np.concatenate([np.arange(130), rng.integers(0, M, 800), np.arange(M - 130, M)]))
    got = to_np(out[torch.from_numpy(rows).to(DEV)])
    ref = sum(_bf(x[rows]) @ _bf(y) for x, y in zip(a, w))
    mag = sum(np.abs(_bf(x[rows])) @ np.abs(_bf(y)) for x, y in zip(a, w))
    assert np.all(np.abs(got - ref) <= (K + K2 + 2) * 2.0 ** -24 * mag + 2.0 ** -8 * np.abs(ref) + 1e-30)


@pytest.mark.parametrize("M,K,K2,N", [
    (23999, 64, 0, 128), (24000, 64, 0, 128), (39999, 100, 0, 113), (40000, 100, 0, 113), (74999, 191, 0, 128),
    (75000, 191, 0, 128), (100000, 128, 0, 120), (299999, 72, 0, 128), (300000, 72, 0, 128), (699999, 20, 0, 128),
    (700000, 20, 0, 128), (349999, 224, 0, 128), (350000, 224, 0, 128), (449999, 193, 0, 96), (450000, 193, 0, 96),
    (450000, 192, 0, 112), (450003, 192, 0, 128), (450000, 255, 0, 81), (8999, 70, 0, 256), (9000, 70, 0, 256),
    (12001, 128, 128, 250), (32767, 100, 0, 208), (32768, 100, 0, 208), (39999, 128, 0, 200), (40000, 128, 0, 200),
    (149999, 65, 0, 180), (150000, 65, 0, 180), (74999, 192, 0, 207), (75000, 192, 0, 207), (399999, 64, 128, 120),
    (400000, 64, 128, 120), (65001, 128, 0, 209)])
def test_lines_between_the_kernels(M, K, K2, N):
    """Both sides of where streamed weights, 128-column tiles and resident weights
    take over from each other; a workspace of the size asked for serves all."""
    g = torch.Generator(device=DEV).manual_seed(M + K + K2 + N)

    def rows16(k):
        a = torch.randn(M, (k + 7) // 8 * 8, generator=g, device=DEV).to(torch.bfloat16)
        a[:, k:] = float("nan")
        return a[:, :k]

    a = [rows16(k) for k in (K, K2) if k]
    w = [(torch.rand(k, N, generator=g, device=DEV) * 2 - 1).to(torch.bfloat16) for k in (K, K2) if k]
    op = S.saga_gemm_op()
    op.dtype, op.mode = S.SAGA_BF16, S.SAGA_GEMM_CONCAT if K2 else S.SAGA_GEMM_PLAIN
    out = S.padded_empty(M, N, torch.bfloat16, DEV)
    out.fill_(float("nan"))
    ws = S.workspace(S.saga_apply_vertex_workspace_size(op, K, K2, N), DEV)
    print(f"lines {M} x {K}+{K2} x {N}", flush=True)
    S.saga_apply_vertex(op, S.cmat(a[0]), S.cmat(w[0]), S.cmat(a[1] if K2 else None), S.cmat(w[1] if K2 else None),
                        None, None, S.mat(out), S._ptr(ws), ws.numel(), S.stream_handle())
    assert not bool(torch.isnan(out).any())
    rows = torch.cat([torch.arange(130), torch.randint(M, (800,)), torch.arange(M - 130, M)]).to(DEV)
    got = to_np(out[rows])
    ref = sum(to_np(x[rows]) @ to_np(y) for x, y in zip(a, w))
    mag = sum(np.abs(to_np(x[rows])) @ np.abs(to_np(y)) for x, y in zip(a, w))
    assert np.all(np.abs(got - ref) <= (K + K2 + 2) * 2.0 ** -24 * mag + 2.0 ** -8 * np.abs(ref) + 1e-30)
