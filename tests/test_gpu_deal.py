"""The sizes of matching work items, and one launch for both levels or one each, by a call's
size: on either side of each line the results are those of items of one group per wave and
one launch per level, bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2604_07980_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# (frames, H, W, boxes of a frame, vertical range): boxes x pixels about 0.1, 0.33, 0.66 and
# 1.0 (one frame), 0.6, 0.8 and 2.1 billion (batches), and 0.5 and 1.0 with a vertical range
@pytest.mark.parametrize("n, h, w, boxes, dy", [
    (1, 2160, 3840, 12, 0), (1, 2160, 3840, 40, 0), (1, 2160, 3840, 80, 0), (1, 2160, 3840, 120, 0),
    (4, 1201, 1917, 65, 0), (4, 1201, 1917, 87, 0), (8, 1201, 1917, 115, 0),
    (1, 2160, 3840, 60, 1), (1, 2160, 3840, 120, 1)])
def test_sizes_change_no_result(lib, n, h, w, boxes, dy):
    rng = np.random.default_rng(n * 1000 + boxes)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(boxes)
    frames, rows = [], []
    for _ in range(n):
        left = torch.randint(0, 256, (h, w), dtype=torch.uint8, device=DEV, generator=gen)
        frames.append((left, torch.roll(left, -21, 1).contiguous(), boxes))
        side = np.exp(rng.uniform(np.log(12), np.log(400), (boxes, 2))).astype(np.int64)
        x0, y0 = rng.integers(0, w - 12, boxes), rng.integers(0, h - 12, boxes)
        rows.append(np.stack([x0, y0, x0 + side[:, 0], y0 + side[:, 1], rng.random(boxes) < 0.8], 1))
    bx = torch.from_numpy(np.concatenate(rows).astype(np.int32)).to(DEV)
    p = synth.base_params()
    p.update(dy_min=-dy, dy_max=dy)

    def run(**options):
        # a context of its own, in which no option was set
        h_ = C.c_void_p()
        assert lib.load().ocsr_ctx_create(0, C.byref(h_)) == lib.OK
        lib.context(0)
        shared, lib._ctx[0] = lib._ctx[0], h_
        try:
            for k, v in options.items():
                lib.set_option(getattr(lib, k), v)
            out = lib.range_batch(frames, bx, p).cpu().numpy()
        finally:
            lib._ctx[0] = shared
            lib.load().ocsr_ctx_destroy(h_)
        return out

    got = run()
    assert (got == run(OPTION_BLOCKS_PER_WAVE=1, OPTION_LEVEL_LAUNCHES=1)).all()
    assert got[:, 2].any()                      # some boxes are ranged


# (frames, H, W): 5 and 3 tiles per resident slot of 256 compute units (7 slots each) from
# four and eight frames on are 8960 and 5376 tiles; just below and above them
@pytest.mark.parametrize("n, h, w", [(4, 928, 1920), (4, 1056, 1920), (8, 544, 900), (8, 608, 1000), (3, 1200, 1920)])
def test_listed_census_changes_no_result(lib, n, h, w):
    rng = np.random.default_rng(n * h)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(w)
    frames, rows = [], []
    for k in range(n):
        left = torch.randint(0, 256, (h - k, w), dtype=torch.uint8, device=DEV, generator=gen)
        frames.append((left, torch.roll(left, -13, 1).contiguous(), 20))
        side = rng.integers(12, 200, (20, 2))
        x0, y0 = rng.integers(-5, w - 12, 20), rng.integers(-5, h - 12, 20)
        rows.append(np.stack([x0, y0, x0 + side[:, 0], y0 + side[:, 1], rng.random(20) < 0.8], 1))
    bx = torch.from_numpy(np.concatenate(rows).astype(np.int32)).to(DEV)
    p = synth.base_params()
    try:
        got = lib.range_batch(frames, bx, p).cpu().numpy()
        lib.set_option(lib.OPTION_CENSUS_TILE_LIST, 0)
        assert (got == lib.range_batch(frames, bx, p).cpu().numpy()).all()
    finally:
        lib.set_option(lib.OPTION_CENSUS_TILE_LIST, 1)
    assert got[:, 2].any()
