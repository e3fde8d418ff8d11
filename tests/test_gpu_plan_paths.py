"""The plan's arrays, whole numbers, at the sizes where its kernels change:
tiles of the degree order, digits of the largest in-degree, the direct and the
tile-sorted out-degree count."""
import numpy as np
import pytest

from gpu_util import graph

pytestmark = pytest.mark.gpu


def _plan(rp, col, num_src, T, B, c=4):
    """include/saga.h's definition of the plan arrays."""
    d = np.diff(rp)
    V = d.shape[0]
    perm = np.argsort(-d, kind="stable")
    dp = d[perm]
    ns = np.where(dp > T, -(-dp // T), 1)
    first = np.concatenate([[0], np.cumsum(ns)])
    pos = np.repeat(np.arange(V), ns)
    j = np.arange(pos.shape[0]) - first[pos]
    beg = rp[perm[pos]] + j * T
    end = np.minimum(beg + T, rp[perm[pos] + 1])
    end = np.where(dp[pos] > T, end, rp[perm[pos] + 1])
    P = np.concatenate([[0], np.cumsum(end - beg + c)])[:-1]
    blk = P // B
    ptr = np.searchsorted(blk, np.arange(blk[-1] + 2))
    return dict(d_in=d, d_out=np.bincount(col, minlength=num_src), perm=perm, row_seg_first=first,
                seg_row=perm[pos], seg_beg=beg, seg_end=end, block_ptr=ptr), dp, T


def _check(deg, num_src, seg_len, block_cost, seed=0):
    deg = np.asarray(deg, dtype=np.int64)
    rp = np.concatenate([[0], np.cumsum(deg)])
    col = np.random.default_rng(seed).integers(0, num_src, rp[-1])
    g = graph(rp, col, num_src=num_src, seg_len=seg_len, block_cost=block_cost)
    ref, dp, T = _plan(rp, col, num_src, seg_len, block_cost)
    got = g.arrays()
    for k, r in ref.items():
        assert np.array_equal(got[k].cpu().numpy(), r), k
    n_split = int((dp > T).sum())
    assert g.counts.n_split == n_split and g.counts.s_split == ref["row_seg_first"][n_split]


@pytest.mark.parametrize("V", [1, 63, 511, 513, 2047, 2048, 2049, 4096, 128 * 2048 - 1, 128 * 2048 + 1,
                               1024 * 2048 - 1, 1024 * 2048 + 1])
def test_tiles(V):
    """Rows per tile, the scan inside the scatter (128 tiles), the sums added
    up by each workgroup (4096 tiles of 512); a split row at either end of a tile."""
    deg = np.random.default_rng(V).integers(0, 4, V)
    deg[:: max(1, V // 3)] = 40
    _check(deg, V, 8, 64)


@pytest.mark.parametrize("hub", [255, 256, 300, 65535, 65536, 70000])
def test_degree_digits(hub):
    """Passes of the degree sort that run: one up to 255, two up to 65535."""
    deg = np.random.default_rng(hub).integers(0, 300 if hub > 300 else 200, 5000)
    deg[[7, 4999]] = hub, max(0, hub - 1)
    _check(deg, 5000, 128, 1024)


@pytest.mark.parametrize("num_src,E", [(1, 5), (16384, 3000), (16385, 70000), (131072, 32 * 1024 * 1024),
                                       (131072, 32 * 1024 * 1024 + 1), (131073, 3728270), (131073, 3728271)])
def test_out_degree_paths(num_src, E):
    """One bucket, several, and both sides of the direct count's limit."""
    V = 1000
    deg = np.full(V, E // V)
    deg[3] += E - deg.sum()
    _check(deg, num_src, 512, 4096)


@pytest.mark.parametrize("num_src,E", [(50, 4000), (131072 * 3, 12000000)])
def test_a_bad_source_id_does_not_reach_the_row_order(num_src, E):
    """Out-degrees and row order may run on two streams: an id out of range,
    found by the former, changes nothing in the latter and is what is reported."""
    from gpu_util import lib

    S, V, T, B = lib(), 700, 64, 256
    deg = np.full(V, E // V)
    deg[5] += E - deg.sum()
    rp = np.concatenate([[0], np.cumsum(deg)])
    col = np.random.default_rng(1).integers(0, num_src, E)
    ref, _, _ = _plan(rp, col, num_src, T, B)
    col[E // 2] = num_src
    g = graph(rp, col, num_src=num_src, seg_len=T, block_cost=B, check=False)
    st, g.counts = S.saga_plan_check(g.plan, S.stream_handle())
    assert st == S.SAGA_EGRAPH and g.counts.error_flags == 8
    got = g.arrays()
    for k in ("d_in", "perm", "row_seg_first", "seg_row", "seg_beg", "seg_end", "block_ptr"):
        assert np.array_equal(got[k].cpu().numpy(), ref[k]), k


def test_a_bad_graph_is_reported_ahead_of_a_broken_invariant():
    from gpu_util import lib

    S = lib()
    g = graph([0, 1, 2], [1, 0])
    for flags, status in ((8 | 1 << 16, S.SAGA_EGRAPH), (1 << 16, S.SAGA_EINTERNAL)):
        g._view(g.plan.counts, 8)[4] = flags
        assert S.saga_plan_check(g.plan, S.stream_handle())[0] == status
