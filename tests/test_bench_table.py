"""Which rows of bench.py's kernel table are given a fraction of the HBM peak."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

BYTES = {"viterbi": 2.0e9, "forward": 2.0e9, "backward": 2.0e9, "counts": 1.0e9, "scores": 4.0e9, "grad_fill": 2.0e9}


def _table(slow):
    """Ten steps; passes over lists take 0.1 ms a pass, or 1 ms (their rate on dense bytes is then below the peak)."""
    ms = 1.0 if slow else 0.1
    prof = {k: (10 * (ms if k not in ("scores", "grad_fill") else 1.0), 10) for k in BYTES}
    return bench.kernel_table(prof, BYTES, 10)


def test_passes_over_lists_get_no_fraction_at_any_rate():
    for slow in (False, True):
        t = _table(slow)
        for k in ("viterbi", "forward", "backward", "counts"):
            assert t[k]["alg_frac"] is None, (k, slow)
        assert t["scores"]["alg_frac"] == 0.5
        assert t["grad_fill"]["alg_frac"] == 0.25
        total = 4 * (1.0 if slow else 0.1) + 2.0
        assert abs(bench.moved_frac(t, 10, total) - 6.0e9 / (total * 1e-3) / 1e9 / bench.PEAK_HBM_GBS) < 1e-4
        only = {k: v for k, v in t.items() if k in ("viterbi", "forward")}
        assert bench.roofline_of(only)["bound"] == "latency" and bench.roofline_of(only)["frac"] is None
        assert bench.moved_frac(only, 10, 1.0) is None


def test_count_path_that_ran():
    t = {"threads_per_sentence": 256, "count_path": "records", "times": {}}
    assert "fixed_point" in bench.tuned_of(t)["counts_taken"] and "times" not in bench.tuned_of(t)
    assert "counts_taken" not in bench.tuned_of({**t, "count_path": "grouped"})
