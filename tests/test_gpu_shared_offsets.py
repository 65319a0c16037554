"""Vertical offsets of a group of blocks shared by a workgroup's waves (calls of at most 2048 groups
with one group to a wave) or walked by one wave (two groups to a wave are never shared): numbers
of offsets below, at and above the four waves, blocks of every matcher, crowded and ineligible
ones, several frames, and calls on both sides of the line. Records are the oracle's."""
import numpy as np
import pytest
import torch

from paper_2604_07980_amd import synth
from test_gpu_parity import _check_debug, _cuda, _gpu_levels, assert_results_match

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dy", [(0, 1), (-1, 1), (-1, 2), (-2, 2), (3, 3), (-4, 4)], ids=lambda d: f"dy{d[0]}_{d[1]}")
@pytest.mark.parametrize("far, fd, close, cd", [(4, 32, 8, 64), (8, 48, 8, 96), (4, 100, 4, 64), (4, 190, 8, 33)])
def test_shared_offsets(lib, orc, far, fd, close, cd, dy):
    H, W = 130, 260
    rng = np.random.default_rng(far + fd + close + cd)
    left, right = synth.render_pair(rng, H, W, [(10, 5, 150, 90, 9.0), (90, 40, 250, 125, 15.0)])
    right[70:] = rng.integers(0, 256, (H - 70, W), dtype=np.uint8)      # no match here: blocks disagree
    n = 70
    wh = rng.integers(6, 60, (n, 2))
    x0, y0 = rng.integers(-6, W - 8, n), rng.integers(-6, H - 8, n)
    boxes = np.stack([x0, y0, x0 + wh[:, 0], y0 + wh[:, 1], rng.random(n) < 0.8], 1).astype(np.int32)
    p = synth.base_params()
    p.update(tau_s=30, n_min=1, min_point_pct=60, dy_min=dy[0], dy_max=dy[1],
             far=dict(mode=0, bw=far, bh=far, n_side=8, dmin=0, dmax=fd - 1),
             close=dict(mode=0, bw=close, bh=close, n_side=8, dmin=0, dmax=2 * cd - 1))
    _, (res, blk, cf, cb, nb) = orc.run_scene(left, right, p, boxes, debug=True)
    g = _gpu_levels(lib, left, right, p)
    out, extra = lib.match_boxes(*g, _cuda(boxes), p, debug=True, cap_blocks=nb + 3)   # (never shared)
    assert_results_match(lib.results_to_numpy(out), res)
    _check_debug(lib, extra, blk, cf, cb, nb)
    try:
        for mode in (0, 1):                         # one launch for both levels, and one each
            lib.set_option(lib.OPTION_LEVEL_LAUNCHES, mode)
            for bpw in (0, 1, 2):
                lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, bpw)
                assert (lib.match_boxes(*g, _cuda(boxes), p, cap_blocks=nb + 3) == out).all(), (mode, bpw)
    finally:
        lib.set_option(lib.OPTION_LEVEL_LAUNCHES, 0)
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 0)


# about 0.3, 1, 2 and 3 thousand groups in three frames
@pytest.mark.parametrize("boxes", [8, 24, 50, 80])
def test_both_sides_of_the_line(lib, boxes):
    H, W, n = 400, 700, 3
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(boxes)
    rng = np.random.default_rng(boxes)
    frames, rows = [], []
    for _ in range(n):
        left = torch.randint(0, 256, (H, W), dtype=torch.uint8, device="cuda:0", generator=gen)
        frames.append((left, torch.roll(left, (1, -11), (0, 1)).contiguous(), boxes))
        side = rng.integers(12, 130, (boxes, 2))
        x0, y0 = rng.integers(0, W - 12, boxes), rng.integers(0, H - 12, boxes)
        rows.append(np.stack([x0, y0, x0 + side[:, 0], y0 + side[:, 1], np.ones(boxes, int)], 1))
    bx = torch.from_numpy(np.concatenate(rows).astype(np.int32)).cuda()
    p = synth.base_params()
    p.update(dy_min=-2, dy_max=2, close=dict(p["close"], dmax=95))
    got = lib.range_batch(frames, bx, p).cpu().numpy()
    try:
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 2)
        assert (got == lib.range_batch(frames, bx, p).cpu().numpy()).all()
    finally:
        lib.set_option(lib.OPTION_BLOCKS_PER_WAVE, 0)
    assert got[:, 2].any()
