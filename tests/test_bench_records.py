"""The benchmark's one-launch entry holds figures of that form or none. No GPU."""
import importlib.util
import os

from paper_2604_07980_amd import build

spec = importlib.util.spec_from_file_location("bench", os.path.join(build.ROOT, "bench.py"))
bench = importlib.util.module_from_spec(spec)
spec.loader.exec_module(bench)


def test_one_launch_record():
    ran = {"reset": {"launches": 10, "avg_us": 1.0}, "fused": {"launches": 10, "avg_us": 310.0}}
    assert bench.one_launch_record(0.33333, True, ran) == {"ms_per_batch": 0.3333, "identical": True,
                                                           "kernel_us": 310.0}
    # the call took the multi-launch path: its time is not this form's
    assert bench.one_launch_record(0.1324, True, {}) == {"ms_per_batch": None, "identical": None,
                                                         "kernel_us": None}
