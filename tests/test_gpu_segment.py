"""Segment median by bins: the longest run of block disparities with gaps below tau_d, for
thresholds from 0 (every value a run of its own; values are then sorted) over ones whose
bins just fit to ones above the whole range, boxes from one block to more than the
aggregation keeps in LDS, and views that agree, agree in parts or not at all. The result
is one of the block values or the mean of two, so it equals the oracle's to the parity
tolerance, and the run's length exactly."""
import numpy as np
import pytest

from paper_2604_07980_amd import synth
from test_gpu_parity import _cuda, assert_results_match

pytestmark = pytest.mark.gpu

H, W = 260, 420


def _views(kind, rng):
    if kind == "noise":
        return tuple(rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    planes = [(0, 0, W, H, 3.3)] if kind == "plane" else \
        [(20 + 60 * k, 10, 90 + 60 * k, H - 10, 2.0 + 4.7 * k) for k in range(6)]
    return synth.render_pair(rng, H, W, planes)


@pytest.mark.parametrize("tau", [0.0, 1e-3, 0.078, 0.0785, 0.3, 1.0, 2.0, 40.0, 1e6])
@pytest.mark.parametrize("kind", ["plane", "planes", "noise"])
def test_segment_median(lib, orc, kind, tau):
    rng = np.random.default_rng(7)
    left, right = _views(kind, rng)
    boxes = np.array([[0, 0, W, H, 1], [10, 10, 14, 14, 1], [5, 5, 25, 17, 1], [30, 30, 300, 200, 1],
                      [100, 20, 164, 84, 1], [60, 0, 380, 60, 1]], np.int32)
    for n_min in (1, 3):
        p = synth.base_params()
        p.update(tau_s=1 << 20, agg_mode=0, tau_d=tau, n_min=n_min, lr_tol=32)
        p["far"] = dict(mode=0, bw=4, bh=4, n_side=8, dmin=0, dmax=31)
        want = orc.run_scene(left, right, p, boxes)[1][0]
        assert want["n_valid"][0] > 4096       # more than the aggregation keeps in LDS
        got = lib.results_to_numpy(lib.range_frame(_cuda(left), _cuda(right), _cuda(boxes), p))
        assert_results_match(got, want)
