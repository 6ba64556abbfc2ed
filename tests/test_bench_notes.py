"""bench.py says of a figure that the library derives instead of timing that it does:
the first of two sweeps from zero in one launch (4 bytes per cell of the launch's
12, where a sweep of its own has 12 in FP32 and 24 in FP64)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_derived_sweep_from_zero_is_labelled():
    import bench
    n = 64 * 32 * 17
    assert "not timed apart" in bench.split_note("smooth0", 4.0 * n, n)
    assert bench.split_note("smooth0", 12.0 * n, n) is None
    assert bench.split_note("smooth0", 24.0 * n, n) is None
    assert bench.split_note("smooth", 8.0 * n, n) is None
