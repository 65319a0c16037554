"""Blocks of few kept points in the generic matcher: up to four points are walked without a list,
more are listed. GRID blocks of 1, 2 x 2 and 3 x 3 points, occluders that leave any number of
them, and candidate counts at the edges of the lanes' shares; block records and costs are whole
numbers, bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2604_07980_amd import synth
from test_gpu_parity import _check_debug, _cuda, _gpu_levels, assert_results_match

pytestmark = pytest.mark.gpu

H, W = 96, 300


@pytest.mark.parametrize("nd", [1, 16, 17, 32, 64, 65, 130, 256])
@pytest.mark.parametrize("side", [1, 2, 3])
def test_few_points(lib, orc, side, nd):
    rng = np.random.default_rng(side * 1000 + nd)
    left, right = synth.render_pair(rng, H, W, [(20, 5, 200, 80, 0.4 * nd), (100, 30, 280, 90, 0.2 * nd + 1)])
    boxes = []
    for k in range(40):
        x0, y0 = int(rng.integers(-6, W - 6)), int(rng.integers(-6, H - 6))
        boxes.append([x0, y0, x0 + int(rng.integers(2, 70)), y0 + int(rng.integers(2, 40)), int(k % 4 != 3)])
    boxes = np.array(boxes, np.int32)
    p = synth.base_params()
    p.update(tau_s=30, min_point_pct=10, n_min=1, lr_tol=int(rng.integers(0, 3)), agg_mode=0)
    p["far"] = dict(mode=1, bw=8, bh=8, n_side=side, dmin=0, dmax=nd - 1)
    p["close"] = dict(mode=1, bw=8, bh=8, n_side=side, dmin=2, dmax=2 * nd + 1)
    _, (res, blk, cf, cb, n) = orc.run_scene(left, right, p, boxes, debug=True)
    kept = {bin(int(m)).count("1") for m in blk["mask"]}
    assert side == 1 or kept & set(range(2, 5))     # walked without a list
    assert side < 3 or max(kept) > 4                # listed
    g = _gpu_levels(lib, left, right, p)
    out, extra = lib.match_boxes(*g, _cuda(boxes), p, debug=True, cap_blocks=max(n, 1) + 3)
    assert_results_match(lib.results_to_numpy(out), res)
    _check_debug(lib, extra, blk, cf, cb, n)
    assert (lib.match_boxes(*g, _cuda(boxes), p, cap_blocks=max(n, 1) + 3) == out).all()


@pytest.mark.parametrize("close", [(8, 8, 191), (16, 4, 63)])
def test_few_points_beside_a_close_level(lib, orc, close):
    """The far GRID blocks in one launch with the close level's, and by themselves."""
    rng = np.random.default_rng(close[0])
    left, right = synth.render_pair(rng, 200, 400, [(20, 5, 200, 180, 11.0), (150, 30, 380, 190, 37.0)])
    boxes = np.array([[5 * k, 3 * k, 5 * k + 9 + 6 * (k % 9), 3 * k + 8 + 7 * (k % 7), 1] for k in range(40)], np.int32)
    p = synth.base_params()
    p.update(tau_s=30, n_min=1, far=dict(mode=1, bw=8, bh=8, n_side=2, dmin=0, dmax=40))
    p["close"] = dict(mode=0, bw=close[0], bh=close[1], n_side=8, dmin=0, dmax=close[2])
    want = orc.run_scene(left, right, p, boxes)[1][0]
    got = lib.results_to_numpy(lib.range_frame(_cuda(left), _cuda(right), _cuda(boxes), p))
    assert_results_match(got, want)
