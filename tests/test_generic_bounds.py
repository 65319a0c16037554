"""Bounds audit, on the CPU, of the generic matcher's points: its list of kept points in LDS, the
entry past the list's end, the points' split over groups of lanes, the word offsets of every
load, and the points walked without a list. The kernel's index arithmetic is restated and run
over GRID blocks at the edges of what it takes and over masks of every size; the constants it
is restated with are looked up in the source. No GPU."""
import os
import random
import re

import pytest

from paper_2604_07980_amd import build, synth
from test_grid_bounds import GRID_VARIANTS, _plan

SOURCE = open(os.path.join(build.CSRC, "dev_match.hpp")).read()
ROUND = int(re.search(r"void generic_costs\(.*?constexpr int B = (\d+);", SOURCE, re.S).group(1))
LIST = [eval(m) for m in re.findall(r"(?:tmpl|row|x)\[(64 \+ \d+)\];", SOURCE)]
FEW = int(re.search(r"constexpr int kFewPoints = (\d+);", SOURCE).group(1))


def _in_image(img_words, row, col, W, guard):
    """The word that a load reads: `row + col` where the guard holds, else word 0."""
    at = row + col if guard else 0
    assert 0 <= at < img_words
    if guard:
        assert 0 <= col < W


def _audit(g, mask, pitch, dlo, nd, d_f):
    W, words = g["Ws"], pitch * g["Hs"]
    nx, npts = g["nx"], g["nx"] * g["ny"]
    kept = [t for t in range(64) if (mask >> t) & 1]
    n = len(kept)
    assert 1 <= n <= npts <= 64 and all(t < npts for t in kept)
    px, prow = [0] * 64, [0] * 64
    for lane in range(64):
        if lane < npts:
            px[lane] = g["lx0"] + (2 * (lane % nx) + 1) * g["lw"] // (2 * nx)
            prow[lane] = (g["ly0"] + (2 * (lane // nx) + 1) * g["lh"] // (2 * g["ny"])) * pitch
        _in_image(words, prow[lane], px[lane], W, 0 <= px[lane] < W)
    for step, shift in ((-1, 0), (1, d_f)):         # forward, then backward from the match
        x = [px[t] - shift for t in range(64)]
        for t in kept:
            _in_image(words, prow[t], x[t], W, 0 <= x[t] < W)
        seen = {}
        if n <= FEW:
            for kc in range(nd):
                for t in kept[:FEW]:
                    xc = x[t] + step * (dlo + kc)
                    _in_image(words, prow[t], xc, W, 0 <= xc < W)
                    seen[kc] = seen.get(kc, 0) + 1
        else:
            rank = {t: bin(mask & ((1 << t) - 1)).count("1") for t in kept}
            assert sorted(rank.values()) == list(range(n))
            assert n < min(LIST)                    # entry n is in the list's space
            lst = {rank[t]: (prow[t], x[t]) for t in kept}
            ng = 4 if nd <= 16 else 2 if nd <= 32 else 1
            per = 64 // ng
            for lane in (range(64) if ng > 1 else (0, 1, 62, 63)):
                lane_kc, grp = lane % per, lane // per
                for i0 in range(0, n, ROUND * ng):
                    for r in range(4):
                        if 64 * r >= nd:
                            break
                        kc = lane_kc + 64 * r
                        for j in range(ROUND):
                            i = min(i0 + j * ng + grp, n)
                            row, col = lst.get(i, (0, 0))
                            xc = col + step * (dlo + kc)
                            ok = kc < nd and i < n and 0 <= xc < W
                            _in_image(words, row, xc, W, ok)
                            if kc < nd and i < n:
                                seen[kc] = seen.get(kc, 0) + 1
            for lane in range(64 // ng):            # the lanes that store a candidate's cost
                for r in range(4):
                    assert lane + 64 * r >= nd or lane + 64 * r < 256
            if ng == 1:
                seen = {k: v for k, v in seen.items() if k % 64 in (0, 1, 62, 63)}
        assert all(v == n for v in seen.values())   # every kept point once per candidate
        if n <= FEW or nd <= 32:
            assert len(seen) == nd


def _masks(npts, rng):
    full = (1 << npts) - 1
    out = [full, 1, 1 << (npts - 1)]
    for n in range(1, npts + 1):
        out.append(sum(1 << t for t in rng.sample(range(npts), n)))
    return out


@pytest.mark.parametrize("variant", list(GRID_VARIANTS))
def test_listed_points_stay_in_bounds(variant):
    rng = random.Random(5)
    p = synth.base_params()
    p.update({k: (dict(v) if isinstance(v, dict) else v) for k, v in GRID_VARIANTS[variant].items()})
    sc = synth.scene_small(1000 + len(variant), H=120, W=200, n_planes=6)
    H, W = sc.left.shape
    blocks = [g for b in sc.boxes.tolist() for g in [_plan(b, W, H, p)] if g]
    assert blocks
    for g in blocks[:4]:
        for mask in rng.sample(_masks(g["nx"] * g["ny"], rng), 8):
            _audit(g, mask, g["Ws"] + rng.randrange(9), g["dlo"], g["nd"], g["dlo"] + rng.randrange(g["nd"]))


def test_listed_points_of_extreme_blocks():
    rng = random.Random(6)
    p = synth.base_params()
    W, H = 64, 48
    blocks = 0
    for side in (1, 2, 3, 8):
        for dmax in (0, 15, 16, 31, 32, 64, 255):
            p.update(tau_s=1 << 30, far=dict(mode=1, bw=8, bh=8, n_side=side, dmin=0, dmax=dmax))
            for b in ([0, 0, W, H, 1], [3, 4, 4, 5, 1], [60, 40, 90, 90, 1], [10, 10, 14, 40, 1]):
                g = _plan(b, W, H, p)
                if g is None:
                    continue
                blocks += 1
                for mask in rng.sample(_masks(g["nx"] * g["ny"], rng), 2):
                    for d_f in (g["dlo"], g["dlo"] + g["nd"] - 1):
                        _audit(g, mask, g["Ws"] + rng.randrange(3), g["dlo"], g["nd"], d_f)
    assert blocks > 50
