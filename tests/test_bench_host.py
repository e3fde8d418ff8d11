"""Host-side helpers of bench.py (no GPU)."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


def test_spread_nearest_rank_p90():
    v = [float(x) for x in range(20, 0, -1)]      # 20 .. 1, unsorted input
    assert bench.spread(v) == {"median": 10.5, "min": 1.0, "p90": 18.0}
    assert bench.spread([3.0, 1.0, 2.0, 10.0, 4.0]) == {"median": 3.0, "min": 1.0, "p90": 10.0}
    assert bench.spread([float(x) for x in range(1, 11)])["p90"] == 9.0
    assert bench.spread([2.5]) == {"median": 2.5, "min": 2.5, "p90": 2.5}


def test_a_stage_without_work_gets_no_rates():
    """Both gate transforms of the gated layer are one product: its stage carries
    the work of both, the empty one neither work nor rates, whatever its time."""
    import numpy as np

    V, E, F, Fe = 1000, 12000, 64, 16
    g = {"num_vertices": V, "num_edges": E, "H": np.zeros((1, F)), "E_feat": np.zeros((1, Fe))}
    stages = bench.suite_stages("gated_rgg", g)
    assert [s[0] for s in stages[0]] == ["source-gate transform", "destination-gate transform", "gated gather",
                                         "GRU transform"]
    roof = bench.suite_rooflines("gated_rgg", stages, [[[0.03], [0.0], [0.1], [0.05]]])
    assert roof[0]["TFLOPs"] == 2 * V * F * 2 * F / 0.03e-3 / 1e12
    assert roof[0]["compulsory_bytes"] == 4 * (V * F + F * 2 * F + V * 2 * F)
    assert roof[1]["compulsory_bytes"] == 0 and not any("GBps" in k or "TFLOPs" in k for k in roof[1])
    assert all("compulsory_GBps" in roof[k] for k in (0, 2, 3))
