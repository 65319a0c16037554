"""Dense matching of few candidates: up to 8 take the vector ALU kernel, more the products, whose
smallest chunk is 2 (32 - 2R) candidate columns. Widths at the edges of a strip of 64 - 2R
columns, heights at those of a band and of four, and the first and last candidate counts of
each kernel. Whole numbers: bit-exact against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(1, 1, 0, 0), (2, 3, 0, 7), (8, 58, 0, 7), (9, 61, 3, 8), (33, 125, 1, 7), (64, 200, 0, 4),
          (7, 30, 40, 44), (5, 20, 30000, 30006), (17, 66, 0, 8), (9, 90, 2, 17), (33, 59, 0, 30),
          (24, 131, 5, 42), (10, 300, 0, 45)]


def _pair(H, W, seed):
    rng = np.random.default_rng(seed)
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
    return CL, CR, gl, gr


@pytest.mark.parametrize("radius", [1, 2, 3])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_d{s[2]}-{s[3]}")
def test_few_candidates(lib, orc, shape, radius):
    H, W, dmin, dmax = shape
    CL, CR, gl, gr = _pair(H, W, H * 1000 + W)
    want, want_r = orc.dense(CL, CR, dmin, dmax, radius, 1)
    got, got_r = lib.dense(gl, gr, dmin, dmax, radius, 1, right=True)
    got, got_r = got.cpu().numpy(), got_r.cpu().numpy()
    assert (got_r == want_r).all(), np.argwhere(got_r != want_r)[:10]
    assert (got == want).all(), np.argwhere(got != want)[:10]


@pytest.mark.parametrize("dmax", [7, 8])
def test_few_candidates_at_offsets(lib, orc, dmax):
    """Several pairs in one launch: every offset's map is that of its own pair."""
    H, W, n = 19, 70, 3
    CL, CR, gl, gr = _pair(H + 4, W, 5)
    p = dict(roi_x0=0, roi_y0=2, roi_w=W, roi_h=H, delta_min=-1, delta_max=n - 2, dmin=0, dmax=dmax,
             radius=2, lr_tol=1, d_min=2)
    counts, maps = lib.rect_offset_counts(gl, gr, p, with_maps=True)
    counts, maps = counts.cpu().numpy(), maps.cpu().numpy()
    for k in range(n):
        y0 = 2 - (k - 1)
        want, _ = orc.dense(np.ascontiguousarray(CL[y0:y0 + H]), np.ascontiguousarray(CR[2:2 + H]), 0, dmax, 2, 1)
        assert (maps[k] == want).all()
        assert counts[k] == (want > 2).sum()


def test_few_candidates_cost_less(lib):
    """Eight candidates take well below what 64 do (53 against 97 us): they do not pay for a chunk
    of the products."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    gl = torch.randint(-(1 << 62), 1 << 62, (1080, 1920), dtype=torch.int64, device=DEV, generator=g)
    gr = torch.roll(gl, -5, 1).contiguous()
    ws = lib.Workspace()

    def ms(dmax):
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                lib.dense(gl, gr, 0, dmax, 2, 1, workspace=ws)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[4]

    assert ms(7) < 0.75 * ms(63)
