"""The matrix-core matchers at the edges of their tiling: blocks of every side up to 8 (two
per wave) and up to 4 (four per wave), candidate counts at and past a lane's share, boxes
whose block rows end in an incomplete group, strips that leave the image on both sides,
occluded points, and unrelated views, whose random winners put the blocks of a group in
backward passes of their own. Block records, masks and cost vectors are whole numbers:
bit-exact against the oracle (the parity tolerances apply to the sub-pixel values)."""
import numpy as np
import pytest

from paper_2604_07980_amd import synth
from test_gpu_parity import _check_debug, _cuda, _gpu_levels, assert_results_match

pytestmark = pytest.mark.gpu

H, W = 90, 260
# (bw, bh, dmin, dmax) of the far path (level scale 1)
PATHS = [(8, 8, 0, 0), (8, 8, 0, 30), (8, 8, 2, 33), (8, 8, 0, 32), (8, 8, 0, 63), (8, 8, 1, 96),
         (8, 8, 0, 96), (8, 8, 0, 127), (8, 8, 5, 164), (8, 8, 0, 190), (8, 8, 0, 255),
         (5, 8, 0, 40), (8, 3, 0, 95), (7, 1, 0, 70), (1, 8, 0, 31), (6, 5, 3, 20),
         (4, 4, 0, 0), (4, 4, 0, 15), (4, 4, 0, 31), (4, 4, 2, 34), (4, 4, 0, 63), (4, 4, 0, 100),
         (3, 4, 0, 31), (2, 1, 0, 20), (1, 1, 0, 31), (4, 2, 7, 60)]


def _boxes(rng):
    b = [[0, 0, W, H, 1], [3, 4, 3 + 8 * 3 + 6, 60, 1], [120, 10, 120 + 37, 10 + 21, 1],
         [W - 30, 20, W + 20, 70, 1], [-12, 30, 20, 70, 1], [50, 50, 54, 54, 1], [60, 5, 61, 80, 1]]
    for _ in range(5):
        x0, y0 = int(rng.integers(0, W - 20)), int(rng.integers(0, H - 20))
        b.append([x0, y0, x0 + int(rng.integers(9, 90)), y0 + int(rng.integers(9, 50)), int(rng.integers(0, 3) > 0)])
    return np.array(b, np.int32)


@pytest.mark.parametrize("related", [True, False], ids=["pair", "noise"])
@pytest.mark.parametrize("path", PATHS, ids=lambda p: f"{p[0]}x{p[1]}_d{p[2]}-{p[3]}")
def test_matrix_matcher(lib, orc, path, related):
    bw, bh, dmin, dmax = path
    rng = np.random.default_rng(bw * 1000 + bh * 100 + dmax)
    if related:
        left, right = synth.render_pair(rng, H, W, [(20, 5, 200, 80, 0.6 * dmax), (100, 30, 240, 85, 0.3 * dmax + 1)])
    else:
        left, right = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    boxes = _boxes(rng)
    p = synth.base_params()
    p.update(tau_s=1 << 20, min_point_pct=int(rng.integers(1, 80)), lr_tol=int(rng.integers(0, 3)))
    p["far"] = dict(mode=0, bw=bw, bh=bh, n_side=8, dmin=dmin, dmax=dmax)
    _, (res, blk, cf, cb, n) = orc.run_scene(left, right, p, boxes, debug=True)
    g = _gpu_levels(lib, left, right, p)
    out, extra = lib.match_boxes(*g, _cuda(boxes), p, debug=True, cap_blocks=max(n, 1) + 3)
    assert_results_match(lib.results_to_numpy(out), res)
    _check_debug(lib, extra, blk, cf, cb, n)
    plain = lib.match_boxes(*g, _cuda(boxes), p, cap_blocks=max(n, 1) + 3)
    assert (plain == out).all()         # the kernels without debug output


@pytest.mark.parametrize("dy", [(-2, 3), (-6, -1)], ids=lambda d: f"dy{d[0]}_{d[1]}")
@pytest.mark.parametrize("path", [(8, 8, 0, 31), (8, 8, 1, 96), (8, 8, 0, 127), (8, 8, 0, 159), (5, 7, 0, 40),
                                  (4, 4, 0, 31), (4, 4, 0, 63), (4, 4, 0, 100), (3, 2, 5, 9)],
                         ids=lambda p: f"{p[0]}x{p[1]}_d{p[2]}-{p[3]}")
def test_matrix_matcher_vertical(lib, orc, path, dy):
    """The same over a vertical range: unrelated views (every group's blocks at offsets of
    their own) and boxes whose strips leave the image above and below."""
    bw, bh, dmin, dmax = path
    rng = np.random.default_rng(bw * 1000 + bh * 100 + dmax + dy[0])
    left, right = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    right[:, :W // 2] = synth.drift_rows(left, dy[1])[:, W // 8:W // 8 + W // 2]
    boxes = _boxes(rng)
    p = synth.base_params()
    p.update(tau_s=1 << 20, min_point_pct=30, dy_min=dy[0], dy_max=dy[1])
    p["far"] = dict(mode=0, bw=bw, bh=bh, n_side=8, dmin=dmin, dmax=dmax)
    p["close"] = dict(p["close"], dmax=31)
    _, (res, blk, cf, cb, n) = orc.run_scene(left, right, p, boxes, debug=True)
    g = _gpu_levels(lib, left, right, p)
    out, extra = lib.match_boxes(*g, _cuda(boxes), p, debug=True, cap_blocks=max(n, 1) + 3)
    assert_results_match(lib.results_to_numpy(out), res)
    _check_debug(lib, extra, blk, cf, cb, n)
    assert (lib.match_boxes(*g, _cuda(boxes), p, cap_blocks=max(n, 1) + 3) == out).all()
