"""Frames of many boxes: a work item's box is found among the boxes' running item ends, in one
step up to 256 boxes and by narrowing steps of 64 above. Counts at the edges of those steps,
boxes without items (not ranged, empty, past the capacity) among them."""
import numpy as np
import pytest
import torch

from paper_2604_07980_amd import synth
from test_gpu_parity import _cuda, assert_results_match

pytestmark = pytest.mark.gpu


def _boxes(n, H, W, seed):
    rng = np.random.default_rng(seed)
    side = rng.integers(5, 26, (n, 2))
    x0, y0 = rng.integers(-4, W - 8, n), rng.integers(-4, H - 8, n)
    flags = (rng.random(n) < 0.7).astype(np.int64)
    # a stretch of boxes without items, as long as a whole step
    flags[n // 3: n // 3 + min(n // 3, 300)] = 0
    return np.stack([x0, y0, x0 + side[:, 0], y0 + side[:, 1], flags], 1).astype(np.int32)


@pytest.mark.parametrize("n", [255, 256, 257, 320, 4097, 16384, 16385])
def test_results_of_many_boxes(lib, orc, n):
    H, W = (240, 400) if n < 1000 else (600, 1000)
    sc = synth.scene_small(7, H=H, W=W, n_planes=9)
    boxes = _boxes(n, H, W, n)
    p = synth.base_params()
    p.update(tau_s=18, n_min=1)
    want = orc.run_scene(sc.left, sc.right, p, boxes, threads=8)[1][0]
    got = lib.results_to_numpy(lib.range_frame(_cuda(sc.left), _cuda(sc.right), _cuda(boxes), p, cap_blocks=1 << 18))
    assert_results_match(got, want)
    assert want["valid"].sum() > n // 50


@pytest.mark.parametrize("cap", [1, 300])
def test_many_boxes_past_the_capacity(lib, orc, cap):
    """The boxes past the capacity have no items, and the running ends stay where they are."""
    H, W, n = 300, 500, 2000
    sc = synth.scene_small(8, H=H, W=W, n_planes=9)
    boxes = _boxes(n, H, W, 3)
    p = synth.base_params()
    p.update(tau_s=18, n_min=1)
    full = lib.results_to_numpy(lib.range_frame(_cuda(sc.left), _cuda(sc.right), _cuda(boxes), p, cap_blocks=1 << 18))
    got = lib.results_to_numpy(lib.range_frame(_cuda(sc.left), _cuda(sc.right), _cuda(boxes), p, cap_blocks=cap))
    over = got["reason"] == lib.REASONS.index("CAPACITY_OVERFLOW")
    assert over.any()
    assert (got[~over] == full[~over]).all()
