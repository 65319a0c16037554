"""Matching launches of a call with a vertical range: one for both levels by default where such a
kernel is built, always one per level when that is asked for; the results are the same."""
import numpy as np
import pytest

from paper_2604_07980_amd import synth
from test_gpu_parity import _check_debug, _cuda, _gpu_levels, assert_results_match

pytestmark = pytest.mark.gpu


def _call(lib, left, right, boxes, p, mode):
    """The call's results and its number of matching launches."""
    lib.set_option(lib.OPTION_LEVEL_LAUNCHES, mode)
    lib.set_timing(True)
    lib.reset_timing()
    try:
        out = lib.results_to_numpy(lib.range_frame(left, right, boxes, p))
        return out, lib.kernel_time("match")[0]
    finally:
        lib.set_timing(False)
        lib.reset_timing()
        lib.set_option(lib.OPTION_LEVEL_LAUNCHES, 0)


# (far block, far candidates, close block, close candidates): the levels' matchers take two 8 x 8
# blocks per wave or four 4 x 4, up to 32, 64, 96, 128 or 160 and up to 32, 64, 128 or 256
# candidates
@pytest.mark.parametrize("far, fd, close, cd", [
    (4, 32, 8, 96), (4, 32, 8, 32), (8, 32, 8, 32), (8, 64, 8, 64), (8, 96, 8, 33), (8, 128, 8, 160),
    (8, 160, 8, 128), (4, 65, 8, 64), (4, 256, 8, 97), (4, 32, 4, 128), (4, 33, 4, 129), (4, 200, 4, 200),
    (8, 32, 4, 65), (8, 130, 4, 256), (5, 20, 7, 40)])
def test_launches_of_a_vertical_range(lib, orc, far, fd, close, cd):
    rng = np.random.default_rng(far + fd + cd)
    left, right = synth.render_pair(rng, 200, 400, [(20, 5, 200, 180, 11.0), (150, 30, 380, 190, 37.0)])
    boxes = np.array([[7 * k, 4 * k, 7 * k + 12 + 9 * (k % 9), 4 * k + 14 + 11 * (k % 7), int(k % 5 != 4)]
                      for k in range(30)], np.int32)
    p = synth.base_params()
    p.update(tau_s=50, n_min=1, dy_min=-1, dy_max=2)
    p["far"] = dict(mode=0, bw=far, bh=far, n_side=8, dmin=0, dmax=fd - 1)
    p["close"] = dict(mode=0, bw=close, bh=close, n_side=8, dmin=0, dmax=2 * cd - 1)
    want = orc.run_scene(left, right, p, boxes)[1][0]
    assert {int(b) for b in (want["n_blocks"] > 1)} == {0, 1} and want["valid"].any()
    args = _cuda(left), _cuda(right), _cuda(boxes), p
    for mode, launches in ((0, 1), (1, 2), (2, 1)):
        got, n = _call(lib, *args, mode)
        assert n == launches, (mode, n)
        assert_results_match(got, want)


def test_levels_without_a_joint_kernel(lib, orc):
    """Far 4 x 4 blocks over 64 candidates beside close 8 x 8 ones: a launch each in every mode."""
    left, right = synth.render_pair(np.random.default_rng(2), 200, 400, [(20, 5, 200, 180, 11.0)])
    boxes = np.array([[20, 10, 60, 50, 1], [100, 20, 260, 150, 1]], np.int32)
    p = synth.base_params()
    p.update(tau_s=50, n_min=1, dy_min=-1, dy_max=2, far=dict(mode=0, bw=4, bh=4, n_side=8, dmin=0, dmax=63))
    want = orc.run_scene(left, right, p, boxes)[1][0]
    for mode in (0, 1, 2):
        got, n = _call(lib, _cuda(left), _cuda(right), _cuda(boxes), p, mode)
        assert n == 2
        assert_results_match(got, want)


@pytest.mark.parametrize("nd", [65, 128, 129, 256])
@pytest.mark.parametrize("bw, bh", [(4, 4), (3, 2), (1, 1), (4, 1)])
def test_four_small_blocks_over_a_long_range(lib, orc, bw, bh, nd):
    rng = np.random.default_rng(bw * 10 + bh + nd)
    H, W = 60, 420
    left, right = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    right[:, :W // 2] = synth.drift_rows(left, 1)[:, W // 8:W // 8 + W // 2]
    boxes = np.array([[3, 2, 40, 30, 1], [150, 10, 200, 58, 1], [180, 20, 190, 40, 0], [390, 5, 440, 25, 1],
                      [300, 40, 317, 57, 1]], np.int32)
    p = synth.base_params()
    p.update(tau_s=1 << 20, min_point_pct=30, dy_min=-1, dy_max=2)
    p["far"] = dict(mode=0, bw=bw, bh=bh, n_side=8, dmin=0, dmax=nd - 1)
    p["close"] = dict(p["close"], dmax=31)
    _, (res, blk, cf, cb, n) = orc.run_scene(left, right, p, boxes, debug=True)
    g = _gpu_levels(lib, left, right, p)
    out, extra = lib.match_boxes(*g, _cuda(boxes), p, debug=True, cap_blocks=max(n, 1) + 3)
    assert_results_match(lib.results_to_numpy(out), res)
    _check_debug(lib, extra, blk, cf, cb, n)
    assert (lib.match_boxes(*g, _cuda(boxes), p, cap_blocks=max(n, 1) + 3) == out).all()
