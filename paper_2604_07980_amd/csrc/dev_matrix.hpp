// Matching of TILED blocks on the matrix cores (Sec. 4.3.2-4.3.5, Alg. 2): one wave takes a
// group of NB horizontally adjacent blocks of one box, 16 columns in all (two blocks of up
// to 8 x 8 points or four of up to 4 x 4).
//
// A block's cost at disparity d sums, over its rows j and columns i, the Hamming distance of
// CL(x + i, y + j) and CR(x + i - d, y + j). For one image row the distances of the group's 16
// columns to 16 columns of the other view are a 16 x 16 product over the words' 64 bits
// (dev_fp4.hpp); the products of all rows add up in the accumulators, four rows of 32
// digits each a product, so 16 T strip columns take 2 T products per four rows. What is
// left of a block's cost is the sum of its columns i along the diagonal (strip column p + i):
// the accumulators go to LDS as 16-bit sums, one strip column of 16 after the other, and the
// lanes of a block (64 / NB) sum pairs of columns for CPL consecutive candidates each.
//
// The backward search starts at each block's own match, so the group's 16 columns come
// from NB places and the strip covers the union of the blocks' ranges: blocks whose
// ranges start within 16 - BS columns of each other (32 - BS with one more tile) share a
// pass, which neighbouring blocks of one surface do; the others take a pass of their own.
//
// With a vertical range (the census cost over (dx, dy), Sec. 4.3.2) each direction repeats
// the strip for every vertical offset, its rows moved by one, and keeps the costs of the
// offset that has the least so far; blocks share a backward pass when their forward
// offsets are equal too. In calls of few groups the four waves of a workgroup take one group
// together, every fourth offset each, and the least of their keys wins.
//
// Bound: vector ALU (67% busy on a batch) and, between, the latency of each group's own loads.
// Two 8 x 8 blocks and 96 candidates take about 280 instructions and 28 products a direction,
// against 1120 for XORs and popcounts of every term: the close level of 16 x 1200p takes 59 us
// instead of 128. Loading a group's words and strip ahead of its mask or of its digits would
// hide their latency but holds them through code that needs the registers: 24 to 63 spilled,
// and 190 us instead of 130 for that batch.
#pragma once

#include "dev_fp4.hpp"
#include "dev_match.hpp"

namespace ocsr {
namespace dev {

template <int NB, int CPL>
struct Matrix {
  static_assert(NB == 2 || NB == 4, "two 8 x 8 or four 4 x 4 blocks");
  static constexpr int BS = 16 / NB;            // largest block side
  static constexpr int G = BS / 4;              // groups of four rows
  static constexpr int LB = 64 / NB;            // lanes per block in the cost and winner steps
  static constexpr int NC = LB * CPL;           // candidates
  static constexpr int T = NC / 16 + 1;         // tiles of 16 strip columns: NC + 15 are read
  static constexpr int TB = T + 1;              // of a wide backward pass
  // LDS words per strip column: 8 and padding (9 words share a bank among half as many of the
  // lanes of a block, CPL columns apart, where CPL is a multiple of 4)
  static constexpr int VS = NB == 4 && CPL >= 8 ? 9 : 10;
  // V (16 TB columns), then the forward costs of the NB blocks
  static constexpr int kCostAt = 16 * TB * VS;
  static constexpr size_t kLdsBytes = sizeof(uint32_t) * (kCostAt + NB * NC);
  static constexpr float kBias = (float)(kBitsMax * BS);   // keeps a column's sum positive
};

// The point masks and occluders of a group: lane o of co holds the o-th rectangle that may
// hide points of the box (bit o of cand). With more than 64 of them in_lanes is false and
// the frame's boxes are scanned for every group; with more than 64 boxes in the frame and one
// group to a wave that scan is the only one.
__device__ __forceinline__ OccLanes box_occluders(const OccLanes& frame, const MatchWs& ws, int box_off,
                                                  int n, int k, bool one_group, int lane, void* lds) {
  OccLanes oc = frame;
  if (n <= 64) {
    box_candidates(oc, n, k, lane);
    return oc;
  }
  if (one_group) return oc;                     // (in_lanes is false)
  const BoxClip ck = ws.clip[box_off + k];
  BoxClip* list = (BoxClip*)lds;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int cnt = 0;
  for (int jb = 0; jb < n; jb += 256) {
    BoxClip co[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int o = jb + 64 * u + lane;
      co[u] = BoxClip{0, 0, 0, 0};
      if (o < n) co[u] = ws.clip[box_off + o];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int o = jb + 64 * u + lane;
      const bool occ = o < n && o != k && ck.cx0 < co[u].cx1 && co[u].cx0 < ck.cx1 && ck.cy0 < co[u].cy1 &&
                       co[u].cy0 < ck.cy1 && co[u].cy1 > ck.cy1;
      const uint64_t m = __ballot(occ);
      const int at = cnt + (int)__popcll(m & below);
      if (occ && at < 64) list[at] = co[u];
      cnt += (int)__popcll(m);
    }
  }
  wave_sync();
  oc.in_lanes = cnt <= 64;
  if (oc.in_lanes) {
    if (lane < cnt) oc.co = list[lane];
    oc.cand = cnt == 64 ? ~0ull : (1ull << cnt) - 1ull;
  }
  wave_sync();
  return oc;
}

// Whether points (fx + q dx, fy) of box k lie in an occluder, all boxes of the frame scanned for those
// that meet the group's rectangle [bx0, bx1] x [by0, by1] (a crowded frame's boxes have hundreds
// of occluders, a group's rectangle few).
template <int NM>
__device__ __forceinline__ void scan_hidden(const MatchWs& ws, int box_off, int n, int k, int bx0, int bx1,
                                            int by0, int by1, int fx, int dx, int fy, int lane,
                                            bool (&hidden)[NM]) {
  const BoxClip ck = ws.clip[box_off + k];
  for (int jb = 0; jb < n; jb += 256) {
    BoxClip co[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int o = jb + 64 * u + lane;
      co[u] = BoxClip{0, 0, 0, 0};
      if (o < n) co[u] = ws.clip[box_off + o];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int o = jb + 64 * u + lane;
      const bool occ = o < n && o != k && ck.cx0 < co[u].cx1 && co[u].cx0 < ck.cx1 && ck.cy0 < co[u].cy1 &&
                       co[u].cy0 < ck.cy1 && co[u].cy1 > ck.cy1 && co[u].cx0 <= bx1 && co[u].cx1 > bx0 &&
                       co[u].cy0 <= by1 && co[u].cy1 > by0;
      const uint64_t m = __ballot(occ);
#pragma unroll
      for (int q = 0; q < NM; ++q) hidden[q] |= in_lane_rects(m, co[u], fx + q * dx, fy);
    }
  }
}

// Column sums of the group against 16 T (wide: 16 TB) strip columns from x_first on, into
// V[column * VS + group column / 2] as packed 16-bit sums. The strip's rows are y_first .. of
// img; a: the group's digits. Columns outside the image read as 0, and with VERT rows too
// (else every row is inside). Rows past the block's ny (whose points do not count) read row
// ny - 1.
template <class M, bool VERT>
__device__ __forceinline__ void strip_sums(const uint64_t* __restrict__ img, const LevelDev& lv, int x_first,
                                           int y_first, int ny, bool wide, const v4i (&a)[M::G][2],
                                           uint32_t* __restrict__ V, int lane) {
  const int W = lv.W, pitch = lv.pitch;
  constexpr int T = M::T, TB = M::TB, G = M::G;
  const int n = lane & 15, kq = lane >> 4;
  uint64_t w[G][TB];
  if (x_first >= 0 && x_first + 16 * TB <= W && (!VERT || (y_first >= 0 && y_first + ny <= lv.H))) {
    const uint64_t* __restrict__ rows = uniform(img + (size_t)y_first * pitch);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint64_t* p = rows + (size_t)min(kq + 4 * g, ny - 1) * pitch + (x_first + n);
#pragma unroll
      for (int t = 0; t < T; ++t) w[g][t] = p[16 * t];
      if (wide) w[g][T] = p[16 * T];
    }
  } else {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int y = y_first + min(kq + 4 * g, ny - 1);
      const bool y_in = !VERT || (y >= 0 && y < lv.H);
      const uint64_t* p = img + (size_t)(y_in ? y : 0) * pitch;
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const int x = x_first + 16 * t + n;
        const bool ok = y_in && x >= 0 && x < W;
        w[g][t] = p[ok ? x : 0];
        w[g][t] = ok ? w[g][t] : 0ull;
      }
    }
  }
  const uint32_t sign = in_vgpr(kSign);
  v4f acc[TB];
  const float c = 8388608.0f + M::kBias;   // above 2^23 the low bits of the float are the sum
  auto add = [&](int g, int h, int t) {
    acc[t] = mfma_fp4(a[g][h], fp4_bits((uint32_t)(w[g][t] >> (32 * h)), sign, kOne),
                      g == 0 && h == 0 ? v4f{c, c, c, c} : acc[t]);
  };
  auto store = [&](int t) {
    auto bits = [&](int r) { return __float_as_uint(acc[t][r]); };
    uint2 v;
    v.x = __builtin_amdgcn_perm(bits(1), bits(0), 0x05040100u);
    v.y = __builtin_amdgcn_perm(bits(3), bits(2), 0x05040100u);
    uint32_t* to = V + (16 * t + n) * M::VS + 2 * kq;
    if constexpr (M::VS % 2 == 0) *(uint2*)to = v;
    else __builtin_memcpy(to, &v, 8);
  };
  // (tile by tile: a tile's digits live for its own products only. Digit group by digit
  // group, with independent products in a row, spills: 137 against 128 us on the batch)
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int h = 0; h < 2; ++h) add(g, h, t);
  if (wide) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int h = 0; h < 2; ++h) add(g, h, T);
  }
#pragma unroll
  for (int t = 0; t < T; ++t) store(t);
  if (wide) store(T);
}

// cost[c]: block b's sum at strip position off + e0 + c in bits 16 and up (the lower bits are
// of no use). A word of V is the sums of columns i and i + 1 (i even) at one strip column;
// summed along i from position q on, its halves are the even columns' part of position q
// and the odd columns' part of q - 1.
template <class M, int CPL>
__device__ __forceinline__ void diagonal_costs(const uint32_t* __restrict__ V, int b, int first,
                                               uint32_t (&cost)[CPL]) {
  const uint32_t* p = V + first * M::VS + b * (M::BS / 2);
  uint32_t q[CPL + 1];
#pragma unroll
  for (int c = 0; c <= CPL; ++c) {
    q[c] = p[c * M::VS];
#pragma unroll
    for (int i = 2; i < M::BS; i += 2) q[c] += p[(c + i) * M::VS + i / 2];
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c) cost[c] = (q[c] << 16) + q[c + 1];
}

// Minimum over the LB lanes of each block, for every lane of the block.
template <int LB>
__device__ __forceinline__ uint32_t block_min(uint32_t v, int lane) {
  v = row16_min_dpp(v);
  if constexpr (LB == 32) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    v = lane < 32 ? lo : hi;
  }
  return v;
}

// Blocks u .. u + NB - 1 (those below nbx) of block row v of a box. VERT: over the path's
// vertical offsets, else at none.
template <int NB, int CPL, bool VERT>
__device__ __forceinline__ void match_group(const MatchParamsDev& P, const FrameDev& fr, const MatchWs& ws,
                                            const DebugDev& dbg, int f, int level, const ItemRec& r,
                                            int u, int v, const OccLanes& oc, int wave, int lane,
                                            void* lds) {
  using M = Matrix<NB, CPL>;
  constexpr int BS = M::BS, G = M::G, LB = M::LB, NC = M::NC;
  uint32_t* V = (uint32_t*)lds;
  uint32_t* costf = V + M::kCostAt;
  const LevelDev& lv = fr.lv[level];
  const PathDev& ph = P.path[level];
  const int nd = ph.nd, dlo = ph.dlo, dhi = dlo + nd - 1;
  const int ndy = VERT ? ph.ndy : 1, dylo = VERT ? ph.dylo : 0;
  // the offsets that this wave walks: all, or every fourth from its own number on
  const bool share = VERT && r.sub >= 0;
  const int ey0 = share ? wave : 0, ey_step = share ? kItemWaves : 1;
  const int nx = r.bw, ny = r.bh, s = lv.scale;
  const int nb = min(NB, r.nbx - u);
  const int X0 = r.ox + u * nx, Y0 = r.oy + v * ny;
  // points kept (Sec. 4.3.5): bit j BS + i of block b's mask, 64 points per ballot
  constexpr int NM = NB * BS * BS / 64;         // ballots: 2 (a block each) or 1 (four blocks)
  uint64_t mask[NM];
  {
    const int pi = lane & (BS - 1), pj = (lane / BS) & (BS - 1), pb = lane / (BS * BS);
    if (__builtin_expect(oc.in_lanes, 1)) {     // (the scan's code out of the way of the rest)
      const BoxClip co = oc.co;
      const bool occ = ((oc.cand >> lane) & 1ull) && co.cx0 <= s * (X0 + nb * nx - 1) && co.cx1 > s * X0 &&
                       co.cy0 <= s * (Y0 + ny - 1) && co.cy1 > s * Y0;
      const uint64_t m = __ballot(occ);
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int b = q + pb;
        const bool hidden = in_lane_rects(m, co, s * (X0 + b * nx + pi), s * (Y0 + pj));
        mask[q] = __ballot(b < nb && pi < nx && pj < ny && !hidden);
      }
    } else {
      bool hidden[NM] = {};
      scan_hidden<NM>(ws, fr.box_off, fr.n_boxes, r.k, s * X0, s * (X0 + nb * nx - 1), s * Y0, s * (Y0 + ny - 1),
                      s * (X0 + pb * nx + pi), s * nx, s * (Y0 + pj), lane, hidden);
#pragma unroll
      for (int q = 0; q < NM; ++q) mask[q] = __ballot(q + pb < nb && pi < nx && pj < ny && !hidden[q]);
    }
  }
  auto block_mask16 = [&](int b) {              // block b's mask
    if constexpr (NB == 2) return mask[b];
    else return (mask[0] >> (16 * b)) & 0xFFFFull;
  };
  uint32_t eligible = 0;                        // bit b
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int pts = (int)__popcll(block_mask16(b));
    if (pts > 0 && 100 * pts >= P.min_point_pct * nx * ny) eligible |= 1u << b;
  }

  // lane roles: group column m and row kq of four (digits); block b, candidates e0 .. (winners)
  const int m = lane & 15, kq = lane >> 4, tb = m / BS, ti = m & (BS - 1);
  const int b = lane / LB, e0 = CPL * (lane & (LB - 1));
  const int slot = f * P.cap_blocks + r.off + v * r.nbx + u + b;
  const bool lead = (lane & (LB - 1)) == 0;
  const bool writer = lead && b < nb && (!share || wave == 0);
  const bool mine = (eligible >> b) & 1u;       // this lane's block is eligible
  uint32_t keep[G];                             // all ones where the lane's point counts
#pragma unroll
  for (int g = 0; g < G; ++g) {
    uint32_t bits;
    if constexpr (NB == 2) {
      const uint64_t mm = tb ? mask[1] : mask[0];
      bits = (uint32_t)(g ? mm >> 32 : mm) >> (8 * kq + ti);
    } else {
      bits = (uint32_t)(mask[0] >> (16 * tb + 4 * kq + ti));
    }
    keep[g] = (bits & 1u) ? 0xFFFFFFFFu : 0u;
  }
  float d_sub = (float)dlo;
  int d_f = dlo, d_b = dlo, dy_f = 0, dy_b = 0, lr_ok = 0;
  if (eligible) {
    // the group's digits from its words t (rows kq + 4 g)
    v4i a[G][2];
    auto digits = [&](const uint64_t (&t)[G]) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const uint32_t ks = kSign & keep[g], k1 = kOne & keep[g], k2 = kTwo & keep[g], k4 = kFour & keep[g];
        a[g][0] = fp4_fixed((uint32_t)t[g], ks, k1, k2, k4);
        a[g][1] = fp4_fixed((uint32_t)(t[g] >> 32), ks, k1, k2, k4);
      }
    };
    // debug output: a block's sums lack a part that depends on its template words alone
    const bool want_costs = dbg.cost_fwd || dbg.cost_bwd;
    auto rest = [&](const uint64_t (&t)[G]) {
      int q = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) q += keep[g] ? fp4_fixed_rest(t[g]) : 0;
#pragma unroll
      for (int o = 1; o < BS; o <<= 1) q += __shfl_xor(q, o, 64);
      q += __shfl_xor(q, 16, 64);
      q += __shfl_xor(q, 32, 64);
      return __shfl(q, b * BS, 64) - BS * (int)M::kBias;
    };
    const int bg = r.off + v * r.nbx + u + b;   // block number within the frame
    // debug output: the costs kept in LDS as true ones, add: what they lack
    auto put_costs = [&](uint16_t* out, int add) {
      wave_sync();
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int kc = e0 + c;
        if (mine && kc < nd && kc < dbg.cap_nd && bg < dbg.cap_blocks)
          out[(size_t)bg * dbg.cap_nd + kc] = (uint16_t)(((int)costf[b * NC + kc] + add) >> 1);
      }
    };
    uint64_t t[G];
    {
      const uint64_t* __restrict__ Lb = uniform(lv.L + (size_t)Y0 * lv.pitch);
      const int x = X0 + tb * nx + ti;
#pragma unroll
      for (int g = 0; g < G; ++g) t[g] = Lb[keep[g] ? (size_t)(kq + 4 * g) * lv.pitch + x : 0];
    }
    digits(t);
    // forward: strip position q of block 0 is column X0 - dhi + q, candidate e is d = dhi - e.
    // A key is the cost (twice the Hamming sum plus a constant of the block) << 16 | (d - dlo)
    // ndy + (dy - dylo)
    uint32_t cost[CPL];
    uint32_t key = 0xFFFFFFFFu;
    for (int ey = ey0; ey < ndy; ey += ey_step) {
      strip_sums<M, VERT>(lv.R, lv, X0 - dhi, Y0 + dylo + ey, ny, false, a, V, lane);
      wave_sync();
      diagonal_costs<M>(V, b, b * nx + e0, cost);
      uint32_t k = 0xFFFFFFFFu;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int e = e0 + c, kc = nd - 1 - e;
        k = min(k, e < nd ? (cost[c] & 0xFFFF0000u) | (uint32_t)(VERT ? kc * ndy + ey : kc) : 0xFFFFFFFFu);
      }
      k = block_min<LB>(k, lane);
      if (!VERT || k < key) {
        key = k;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int e = e0 + c, kc = nd - 1 - e;
          costf[b * NC + (e < nd ? kc : e)] = cost[c] >> 16;
        }
      }
      if (VERT) wave_sync();
    }
    if (want_costs && dbg.cost_fwd) put_costs(dbg.cost_fwd, rest(t));
    int id = (int)(key & 0xFFFFu);
    int best = VERT ? min(id / ndy, nd - 1) : id;   // (a wave without offsets has no key)
    wave_sync();
    // the parabola's numerator and denominator are both twice those of the Hamming sums, and
    // their quotient the same number
    int ca = (int)costf[b * NC + max(best - 1, 0)];
    int cb = (int)costf[b * NC + min(best + 1, nd - 1)];
    if constexpr (VERT) {
      if (share) {
        // the least key of the four waves, and the costs beside it
        __shared__ uint32_t best_of[kItemWaves][NB][3];
        if (lead) {
          best_of[wave][b][0] = key;
          best_of[wave][b][1] = (uint32_t)ca;
          best_of[wave][b][2] = (uint32_t)cb;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kItemWaves; ++w) {
          const uint32_t k = best_of[w][b][0];
          if (k <= key) {
            key = k;
            ca = (int)best_of[w][b][1];
            cb = (int)best_of[w][b][2];
          }
        }
        id = (int)(key & 0xFFFFu);
        best = id / ndy;
      }
      dy_f = dylo + id - best * ndy;
    }
    d_f = dlo + best;
    if (mine) d_sub = subpixel(d_f, best, nd, ca, (int)(key >> 16), cb);

    // backward: the group's columns are CR(x - d_f) in rows y + dy_f, candidate e of block b is
    // strip column start[b] + e, in rows y + dy_f - dy
    int start[NB], df[NB], ef[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      df[q] = __builtin_amdgcn_readlane(d_f, q * LB);
      ef[q] = VERT ? __builtin_amdgcn_readlane(dy_f, q * LB) : 0;
      start[q] = X0 + q * nx - df[q] + dlo;
    }
    {
      int dt = df[0], et = ef[0];
#pragma unroll
      for (int q = 1; q < NB; ++q) {
        dt = tb == q ? df[q] : dt;
        et = tb == q ? ef[q] : et;
      }
      const uint64_t* __restrict__ Rb = uniform(VERT ? lv.R : lv.R + (size_t)Y0 * lv.pitch);
      const int x = X0 + tb * nx + ti - dt;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int y = (VERT ? Y0 + et : 0) + kq + 4 * g;
        const bool ok = keep[g] && x >= 0 && (!VERT || (y >= 0 && y < lv.H));
        t[g] = Rb[ok ? (size_t)y * lv.pitch + x : 0];
        t[g] = ok ? t[g] : 0ull;
      }
    }
    digits(t);
    uint32_t left = eligible, bkey = 0xFFFFFFFFu;
    if (want_costs) wave_sync();                // the forward costs are read
    while (left) {
      int base = 0x7FFFFFFF, bdy = 0, far = 0;
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (((left >> q) & 1u) && start[q] < base) {
          base = start[q];
          bdy = ef[q];
        }
      uint32_t now = 0;
      int off = 0;
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int o = start[q] - base;
        if (((left >> q) & 1u) && o <= 32 - BS && (!VERT || ef[q] == bdy)) {
          now |= 1u << q;
          far = max(far, o);
          off = b == q ? o : off;
        }
      }
      left &= ~now;
      const bool here = (now >> b) & 1u;
      for (int ey = ey0; ey < ndy; ey += ey_step) {
        strip_sums<M, VERT>(lv.L, lv, base, VERT ? Y0 + bdy - dylo - ey : Y0, ny, far > 16 - BS, a, V, lane);
        wave_sync();
        diagonal_costs<M>(V, b, off + e0, cost);
        uint32_t k = 0xFFFFFFFFu;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int e = e0 + c;
          k = min(k, here && e < nd ? (cost[c] & 0xFFFF0000u) | (uint32_t)(VERT ? e * ndy + ey : e) : 0xFFFFFFFFu);
        }
        if (VERT || want_costs) k = block_min<LB>(k, lane);
        if (want_costs && k < bkey) {
#pragma unroll
          for (int c = 0; c < CPL; ++c) costf[b * NC + e0 + c] = cost[c] >> 16;
        }
        bkey = min(bkey, k);
        wave_sync();
      }
    }
    if (!VERT) bkey = block_min<LB>(bkey, lane);
    if constexpr (VERT) {
      if (share) {
        __shared__ uint32_t bkey_of[kItemWaves][NB];
        if (lead) bkey_of[wave][b] = bkey;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kItemWaves; ++w) bkey = min(bkey, bkey_of[w][b]);
      }
    }
    if (want_costs && dbg.cost_bwd) put_costs(dbg.cost_bwd, rest(t));
    const int bid = (int)(bkey & 0xFFFFu);
    const int bb = VERT ? bid / ndy : bid;
    d_b = dlo + bb;
    if (VERT) dy_b = dylo + bid - bb * ndy;
    lr_ok = mine && abs(d_b - d_f) <= P.lr_tol;   // consistency on d only (Sec. 4.3.3)
  }
  if (writer) {
    ws.blk_val[slot] = (float)s * d_sub;        // d_full = s * d (Sec. 4.1)
    ws.blk_flag[slot] = (uint8_t)((mine ? 1 : 0) | (lr_ok ? 2 : 0));
  }
  if (dbg.blocks) {
    const int bg = r.off + v * r.nbx + u + b;
    uint64_t mk = block_mask16(0);
#pragma unroll
    for (int q = 1; q < NB; ++q) mk = b == q ? block_mask16(q) : mk;
    uint64_t packed = 0;                        // the record's layout: bit j nx + i
    for (int j = 0; j < ny; ++j)
      packed |= ((mk >> (BS * j)) & ((1ull << nx) - 1ull)) << (j * nx);
    if (writer && bg < dbg.cap_blocks) {
      ocsr_block_record rec;
      rec.box = r.k; rec.level_scale = s; rec.u = u + b; rec.v = v;
      rec.px0 = X0 + b * nx; rec.py0 = Y0; rec.nx = nx; rec.ny = ny;
      rec.mask = packed; rec.eligible = mine;
      rec.d_f = mine ? d_f : dlo; rec.d_b = mine ? d_b : dlo;
      rec.lr_ok = lr_ok; rec.d_sub = d_sub; rec.valid = lr_ok;
      rec.dlo = dlo; rec.nd = nd;
      rec.dy_f = mine ? dy_f : 0; rec.dy_b = mine ? dy_b : 0;
      dbg.blocks[bg] = rec;
    }
  }
}

// Matcher of one level's TILED blocks: wave w of a workgroup takes groups r.first + w,
// r.first + w + 4, ... of an item; or, where the waves share a group's vertical offsets (r.sub >=
// 0), all four take group r.first + r.sub. Everything that decides the way to match_group's
// barriers is the same for the four waves: the item, the box, the group's point masks.
template <int NB, int CPL, bool VERT = false>
struct MatrixMatcher {
  static constexpr size_t kLds = (Matrix<NB, CPL>::kLdsBytes + 15) & ~(size_t)15;
  static constexpr bool kShares = VERT;         // a group's offsets may be shared
  using State = OccLanes;
  static __device__ __forceinline__ State frame_state(const MatchWs& ws, const FrameDev& fr, int lane) {
    return frame_lanes(ws, fr.box_off, fr.n_boxes, lane);
  }
  static __device__ __forceinline__ void run_item(const MatchParamsDev& P, const FrameDev& fr,
                                                  const MatchWs& ws, const DebugDev& dbg, int f,
                                                  int level, const ItemRec& r, int wave, int lane,
                                                  void* lds, const State& st) {
    const OccLanes oc = box_occluders(st, ws, fr.box_off, fr.n_boxes, r.k,
                                      P.item_blocks[level] <= kItemWaves || r.sub >= 0, lane, lds);
    const int ngx = (r.nbx + NB - 1) / NB;      // groups per block row
    const bool share = VERT && r.sub >= 0;
    int g = r.first + (share ? r.sub : wave);
    int v = g / ngx, ug = g - v * ngx;
    for (int j = share ? 0 : wave; j < (share ? 1 : P.item_blocks[level]); j += kItemWaves) {
      if (g < r.ngrp) match_group<NB, CPL, VERT>(P, fr, ws, dbg, f, level, r, NB * ug, v, oc, wave, lane, lds);
      g += kItemWaves;
      ug += kItemWaves;
      while (ug >= ngx) {
        ug -= ngx;
        ++v;
      }
    }
  }
};
// two blocks of up to 8 x 8 points and 32 CPL candidates
template <int CPL>
using PairMatcher = MatrixMatcher<2, CPL>;
// four blocks of up to 4 x 4 points and 16 CPL candidates
template <int CPL>
using QuadMatcher = MatrixMatcher<4, CPL>;

}  // namespace dev
}  // namespace ocsr
