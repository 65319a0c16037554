"""Census tiles whose samples are read as words, and the ones beside them that are not.

A tile off the image's border is staged by unaligned eight-byte loads while all its staged
samples and four more to the right are in the level image; the sizes put the second tile of a
row and the second row of tiles exactly at, and one sample short of, that edge. Exact against
the oracle.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TILE_X, TILE_Y = 64, 32


@pytest.mark.parametrize("short_x", [0, 1])
@pytest.mark.parametrize("short_y", [0, 1])
@pytest.mark.parametrize("scale", [1, 2, 3])
@pytest.mark.parametrize("win", [(3, 4), (2, 2), (4, 3)])
def test_word_tile_edges(lib, orc, win, scale, short_y, short_x):
    sx, sy = win
    words = (TILE_X + 2 * sx + 3) // 4
    ws = TILE_X - sx + 4 * words + 4 - short_x
    hs = TILE_Y - sy + TILE_Y + 2 * sy - short_y
    w, h = scale * ws + scale - 1, scale * hs
    rng = np.random.default_rng(97 * scale + 7 * sx + 2 * short_y + short_x)
    # an odd pitch and an odd start, the image's last byte the buffer's last
    pitch, start = w + 2 + w % 2, 3
    buf = rng.integers(0, 256, size=start + (h - 1) * pitch + w, dtype=np.uint8)
    t = torch.from_numpy(buf).to(DEV).as_strided((h, w), (pitch, 1), start)
    img = np.ascontiguousarray(np.lib.stride_tricks.as_strided(buf[start:], (h, w), (pitch, 1)))
    # saturated values and equal neighbours as well as random ones
    img_q = img & np.uint8(0xC0 if short_x else 0xFF)
    if short_x:
        t.bitwise_and_(0xC0)
    for sentinel in (0, 1):
        want = orc.census(img_q, sx, sy, scale, sentinel)
        got = lib.census(t, sx, sy, scale, sentinel).cpu().numpy().view(np.uint64)
        assert (got == want).all(), np.argwhere(got != want)[:10]
