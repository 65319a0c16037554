"""Work items found from the plan's running ends: frames whose box counts sit at the edges
of the search (64 boxes per ballot, 256 per round), and a batch of such frames, against the
oracle. Box results are whole numbers or fp32 values of single IEEE operations on whole
numbers: the parity tolerances of the other ranging tests apply."""
import numpy as np
import pytest
import torch

from paper_2604_07980_amd import synth
from test_gpu_parity import _cuda, assert_results_match

pytestmark = pytest.mark.gpu

H, W = 200, 320


def _scene(n, seed):
    rng = np.random.default_rng(seed)
    planes = synth.random_boxes(rng, H, W, n, scale=0.2, tau_s=20)
    left, right = synth.render_pair(rng, H, W, planes[:40])
    # every fifth box is not ranged, and runs of boxes outside the image have no items
    boxes = np.array([[*q[:4], int(k % 5 != 3)] for k, q in enumerate(planes)], np.int32)
    boxes[n // 3:n // 3 + n // 8, [0, 2]] += 2 * W
    return left, right, boxes


def _params():
    p = synth.params_for(2)
    p["tau_s"] = 20
    return p


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 600])
def test_frame_items(lib, orc, n):
    left, right, boxes = _scene(n, 50 + n)
    p = _params()
    want = orc.run_scene(left, right, p, boxes)[1][0]
    got = lib.results_to_numpy(lib.range_frame(_cuda(left), _cuda(right), _cuda(boxes), p))
    assert_results_match(got, want)


def test_batch_items(lib, orc):
    p = _params()
    scenes = [_scene(n, 90 + n) for n in (257, 3, 64, 130)]
    want = np.concatenate([orc.run_scene(s[0], s[1], p, s[2])[1][0] for s in scenes])
    frames = [(_cuda(s[0]), _cuda(s[1]), len(s[2])) for s in scenes]
    boxes = _cuda(np.concatenate([s[2] for s in scenes]))
    assert_results_match(lib.results_to_numpy(lib.range_batch(frames, boxes, p)), want)
