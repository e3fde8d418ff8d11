"""The LSTM Gather's step loop at its edges: rows around the depth of the P-row
ring (12 loads ahead of a step, 13 slots) and around the chunks of 1024 ids."""
import numpy as np
import pytest

from gpu_util import graph
from helpers import FP32_TOL, rel_err
from test_gpu_lstm import _ref, run_lstm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [32, 64, 128])
def test_rows_around_the_ring_and_the_id_chunks(H):
    d = np.array(list(range(0, 30)) + [1023, 1024, 1025, 1035, 1036, 1037, 2047, 2048, 2060, 2061])
    n = len(d)
    rng = np.random.default_rng(7 * H)
    rp = np.concatenate([[0], np.cumsum(d)]).astype(np.int32)
    col = rng.integers(0, n, int(rp[-1])).astype(np.int32)
    P = rng.standard_normal((n, 4 * H)).astype(np.float32)
    a = 1.0 / np.sqrt(H)
    W_hh = rng.uniform(-a, a, (H, 4 * H)).astype(np.float32)
    print(f"lstm steps H={H}", flush=True)
    got = run_lstm(graph(rp, col, num_src=n), P, W_hh)
    assert rel_err(got, _ref(rp, col, P, W_hh)) <= FP32_TOL
