"""The counter-derived HBM traffic that bench.py prints as `roofline.traffic` is a constant copied from a tracked
rocprofv3 summary: this test keeps the two from drifting apart (CPU only, reads text files of the repository)."""
import importlib.util
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def load_bench():
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_traffic_constants_are_the_profiles_figures():
    bench = load_bench()
    seen = {}
    for name in ("ctx32k_hbm_traffic_pmc.md", "ragged16_hbm_traffic_pmc.md"):
        text = open(os.path.join(ROOT, "profiles", name)).read()
        for workload, value in re.findall(r"^traffic_bytes_per_launch\[(\w+)\] = (\d+)$", text, flags=re.M):
            seen[workload] = int(value)
    assert seen == bench.VERIFY_TRAFFIC_BYTES


def test_traffic_is_close_to_the_algorithmic_bytes():
    """The figures themselves: a verification launch moves its K + V bytes once, plus a few percent of queries, page
    table, collected log-sum-exps and partial results (re-reads would show up here first)."""
    bench = load_bench()
    assert 1.0 <= bench.VERIFY_TRAFFIC_BYTES["ctx32k"] / (32768 * 4096) <= 1.05
    text = open(os.path.join(ROOT, "profiles", "ragged16_hbm_traffic_pmc.md")).read()
    kv = int(re.search(r"K \+ V = ([\d,]+) bytes", text).group(1).replace(",", ""))
    assert 1.0 <= bench.VERIFY_TRAFFIC_BYTES["ragged16"] / kv <= 1.05


def test_phase_table_leaves_out_events_that_a_wave_never_reached():
    """Two workgroups of four waves; a wave without a tile has no first one, and its stamp stays zero: the phases that need it are
    summed up over the others, and a workgroup's XCD has the mean of the waves that streamed."""
    import numpy as np
    import torch
    bench = load_bench()
    rec = np.zeros((16, 8), dtype=np.uint64)                     # the second half: never written
    for w in range(8):
        rec[w] = 10 ** 16 + 100 * np.arange(8, dtype=np.uint64) + 10 * w
    rec[3, 4] = rec[7, 4] = 0
    rec[3, 5] = rec[7, 5] = 10 ** 16 + 350                       # (streamed nothing, long before the others)
    t = bench.timeline_table(torch.from_numpy(rec.view(np.int64)), "kernel", 4)
    assert t["waves"] == 8
    first = t["events_after_first_entry"]["first tile done"]
    assert abs(first["min"] - 4.0) < 0.05 and abs(first["max"] - 4.6) < 0.05
    for phase in ("queries in LDS (first barrier passed) -> first tile done", "first tile done -> last tile done"):
        s = t["phase_durations_per_wave"][phase]
        assert all(abs(s[k] - 1.0) < 0.05 for k in ("min", "p50", "p90", "max")), (phase, s)
    means = t["last_tile_done_mean_by_xcd"]
    assert abs(means[0] - 5.1) < 0.05 and abs(means[1] - 5.5) < 0.05 and means[2:] == [None] * 6
