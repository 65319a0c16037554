"""Matching launches of a call with a vertical range: one for both levels by default where such a
kernel is built, always one per level when that is asked for; the results are the same."""
import numpy as np
import pytest

from paper_2604_07980_amd import synth
from test_gpu_parity import _cuda, assert_results_match

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


# (far block, far candidates, close candidates)
@pytest.mark.parametrize("far, fd, cd", [(4, 32, 96)])
def test_launches_of_a_vertical_range(lib, orc, far, fd, cd):
    rng = np.random.default_rng(far + fd + cd)
    left, right = synth.render_pair(rng, 200, 400, [(20, 5, 200, 180, 11.0), (150, 30, 380, 190, 37.0)])
    boxes = np.array([[7 * k, 4 * k, 7 * k + 12 + 9 * (k % 9), 4 * k + 14 + 11 * (k % 7), int(k % 5 != 4)]
                      for k in range(30)], np.int32)
    p = synth.base_params()
    p.update(tau_s=50, n_min=1, dy_min=-1, dy_max=2)
    p["far"] = dict(mode=0, bw=far, bh=far, n_side=8, dmin=0, dmax=fd - 1)
    p["close"] = dict(p["close"], dmax=2 * cd - 1)
    want = orc.run_scene(left, right, p, boxes)[1][0]
    assert {int(b) for b in (want["n_blocks"] > 1)} == {0, 1} and want["valid"].any()
    args = _cuda(left), _cuda(right), _cuda(boxes), p
    for mode, launches in ((0, 1), (1, 2), (2, 1)):
        got, n = _call(lib, *args, mode)
        assert n == launches, (mode, n)
        assert_results_match(got, want)
