"""Crowded frames: more boxes than a wave has lanes, and boxes with more occluders than that. The
occluders of a group of blocks come from the lanes, from a list made per work item, or from a
scan of the frame's boxes per group; masks, records and results against the oracle."""
import numpy as np
import pytest

from paper_2604_07980_amd import synth
from test_gpu_parity import _check_debug, _cuda, _gpu_levels, assert_results_match

pytestmark = pytest.mark.gpu


# boxes, their largest side, the share of points that has to be visible
@pytest.mark.parametrize("n, side, pct", [(64, 60, 0), (65, 60, 50), (257, 25, 50), (300, 60, 0), (300, 60, 100),
                                          (600, 90, 20)])
@pytest.mark.parametrize("close", [8, 4])
def test_crowded_frames(lib, orc, n, side, pct, close):
    H, W = 130, 220
    rng = np.random.default_rng(n + side + pct)
    left, right = synth.render_pair(rng, H, W, [(10, 5, 150, 90, 9.0), (90, 40, 215, 125, 15.0)])
    wh = rng.integers(8, side + 1, (n, 2))
    x0, y0 = rng.integers(-6, W - 8, n), rng.integers(-6, H - 8, n)
    boxes = np.stack([x0, y0, x0 + wh[:, 0], y0 + wh[:, 1], rng.random(n) < 0.8], 1).astype(np.int32)
    p = synth.base_params()
    p.update(tau_s=20, n_min=1, min_point_pct=pct, far=dict(mode=0, bw=4, bh=4, n_side=8, dmin=0, dmax=31),
             close=dict(mode=0, bw=close, bh=close, n_side=8, dmin=0, dmax=63))
    _, (res, blk, cf, cb, nb) = orc.run_scene(left, right, p, boxes, debug=True)
    assert (blk["eligible"] == 0).any() and (pct == 100 or (blk["eligible"] == 1).sum() > 20)
    g = _gpu_levels(lib, left, right, p)
    out, extra = lib.match_boxes(*g, _cuda(boxes), p, debug=True, cap_blocks=nb + 3)
    assert_results_match(lib.results_to_numpy(out), res)
    _check_debug(lib, extra, blk, cf, cb, nb)
    try:
        for bpw in (0, 1, 3):                       # one group to a wave, and three
            lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, bpw)
            assert (lib.match_boxes(*g, _cuda(boxes), p, cap_blocks=nb + 3) == out).all()
    finally:
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 0)
