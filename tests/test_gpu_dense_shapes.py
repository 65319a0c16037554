"""The dense matcher's matrix-core kernel at the edges of its tiling: strips of up to
32 - 2R output columns, bands of 8 rows, chunks of 2 (16 T - 2R) candidate columns with
T = 3, 4 or 5, images narrower than a window, the smallest and largest ranges, and a
pitched pair. Winners of both views and the checked map are whole numbers: bit-exact
against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# (H, W, dmin, dmax): one column and row; a window; one strip and one past it; a chunk's
# last candidate and one more for each T; ranges that start beyond the image
SHAPES = [(1, 1, 0, 0), (3, 5, 0, 7), (8, 28, 0, 63), (9, 29, 1, 64), (17, 57, 0, 87),
          (16, 85, 2, 97), (33, 190, 0, 119), (24, 203, 0, 127), (10, 260, 4, 163),
          (31, 400, 0, 255), (7, 30, 40, 60), (5, 20, 30000, 30010)]


@pytest.mark.parametrize("radius", [1, 2, 3])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_d{s[2]}-{s[3]}")
def test_dense_shapes(lib, orc, shape, radius):
    H, W, dmin, dmax = shape
    rng = np.random.default_rng(H * 1000 + W)
    # words of few distinct values, all-zero and all-one among them: ties and extreme costs
    pool = rng.integers(0, 1 << 63, size=6, dtype=np.int64).astype(np.uint64)
    pool = np.concatenate([pool, [np.uint64(0), ~np.uint64(0)]])
    CL, CR = pool[rng.integers(0, 8, (H, W))], pool[rng.integers(0, 8, (H, W))]
    CR[:, : W // 2] = CL[:, W - W // 2:]
    big = torch.zeros((2, H + 2, W + 9), dtype=torch.int64, device=DEV)
    big.fill_(-1)                                   # words around the image that must not count
    gl, gr = big[0, 1:H + 1, 5:W + 5], big[1, 1:H + 1, 5:W + 5]
    gl.copy_(torch.from_numpy(CL.view(np.int64)))
    gr.copy_(torch.from_numpy(CR.view(np.int64)))
    want, want_r = orc.dense(CL, CR, dmin, dmax, radius, 1)
    got, got_r = lib.dense(gl, gr, dmin, dmax, radius, 1, right=True)
    got, got_r = got.cpu().numpy(), got_r.cpu().numpy()
    assert (got_r == want_r).all(), np.argwhere(got_r != want_r)[:10]
    assert (got == want).all(), np.argwhere(got != want)[:10]
