// Device code of the object-centric matching steps (Sec. 4.3.2-4.3.6, Alg. 2), shared by
// the multi-launch kernels (match.hip) and the fused persistent kernel (fused.hip).
//
//   plan_frame        one wave per frame: clip, far/close type (Sec. 4.3.4 type
//                     equation), level box, block grid, block and work-item numbers
//   match_block_tiled one wave per block (match_group of dev_matrix.hpp: per group of blocks):
//                     occluder mask (Sec. 4.3.5), forward Hamming
//                     search (census cost equation), winner-take-all, parabola
//                     (sub-pixel equation), backward search and L/R check (Sec. 4.3.3)
//   aggregate_box     one workgroup per box: longest-segment or trimmed median of the
//                     valid block disparities (Sec. 4.3.4), depth Z = f b / d (Eq. 1)
#pragma once

#include "dev_common.hpp"

namespace ocsr {
namespace dev {

// valid block values of a box that the aggregation keeps in LDS; boxes with more
// blocks aggregate from global memory (the method sets no limit on a box's blocks)
constexpr int kAggMax = 4096;

// ---------------------------------------------------------------------------------
// plan: one wave walks the frame's boxes 64 at a time
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void plan_frame(const MatchParamsDev& P, const FrameDev& fr, int f,
                                           int n_total, const ocsr_box* __restrict__ boxes,
                                           const MatchWs& ws, int lane) {
  const int n = fr.n_boxes;
  const int W = fr.W, H = fr.H;
  int carry = 0, carry0 = 0, carry1 = 0;
  // the next 64 boxes are loaded while the current ones are planned
  ocsr_box next = {};
  if (lane < n) next = boxes[fr.box_off + lane];
  for (int base = 0; base < n; base += 64) {
    const int i = base + lane;
    BoxPlan pl = {};
    BoxClip cl = {0, 0, 0, 0};
    int count = 0;
    const ocsr_box b = next;
    if (i + 64 < n) next = boxes[fr.box_off + i + 64];
    if (i < n) {
      const int cx0 = max(b.x0, 0), cy0 = max(b.y0, 0);
      const int cx1 = min(b.x1, W), cy1 = min(b.y1, H);
      const bool empty = !(cx0 < cx1 && cy0 < cy1);
      if (!empty) cl = BoxClip{cx0, cy0, cx1, cy1};   // empty boxes overlap nothing
      if (!(b.flags & OCSR_BOX_RANGE)) {
        pl.status = OCSR_REASON_NOT_RANGED;
      } else if (empty) {
        pl.status = OCSR_REASON_CLIPPED_EMPTY;
      } else {
        // far/close type (Sec. 4.3.4): FAR iff the longer clipped side is below tau_s
        const bool far_box = max(cx1 - cx0, cy1 - cy0) < P.tau_s;
        const int level = far_box ? 0 : 1;
        const LevelDev& lv = fr.lv[level];
        const PathDev& ph = P.path[level];
        const int s = lv.scale;
        pl.level = level;
        // level pixels whose full-res position s*x lies in the box and whose census
        // is defined
        const int x0 = max(cdiv_nonneg(cx0, s), lv.sx), x1 = min(cdiv_nonneg(cx1, s), lv.W - lv.sx);
        const int y0 = max(cdiv_nonneg(cy0, s), lv.sy), y1 = min(cdiv_nonneg(cy1, s), lv.H - lv.sy);
        if (x1 <= x0 || y1 <= y0) {
          pl.status = OCSR_REASON_NO_ELIGIBLE_BLOCKS;
        } else {
          pl.lx0 = x0; pl.ly0 = y0; pl.lw = x1 - x0; pl.lh = y1 - y0;
          if (ph.mode == OCSR_MODE_TILED) {
            // centred grid of whole blocks; one shrunken block when the box is smaller
            pl.bw = min(ph.bw, pl.lw);
            pl.bh = min(ph.bh, pl.lh);
            pl.nbx = max(1, pl.lw / ph.bw);
            pl.nby = max(1, pl.lh / ph.bh);
            pl.ox = pl.lx0 + (pl.lw - pl.nbx * pl.bw) / 2;
            pl.oy = pl.ly0 + (pl.lh - pl.nby * pl.bh) / 2;
          } else {
            // the whole box is one block sampled on an n_side x n_side grid
            pl.nbx = pl.nby = 1;
            pl.bw = min(ph.n_side, pl.lw);
            pl.bh = min(ph.n_side, pl.lh);
          }
          // the method sets no limit on a box's blocks; only the call's capacity does.
          // A count past the capacity saturates at cap + 1 (the box, and every later box,
          // then passes the capacity), which keeps the prefix in 32 bits.
          const long long nb = (long long)pl.nbx * pl.nby;
          pl.status = -1;
          count = (int)min(nb, (long long)P.cap_blocks + 1);
        }
      }
    }
    // block numbers: prefix over the boxes; a range passing the capacity is dropped
    const int incl = wave_incl_scan(count);
    const int off = carry + incl - count;
    int nblk = 0;
    if (pl.status == -1 && i < n) {
      if ((long long)off + count > (long long)P.cap_blocks) pl.status = OCSR_REASON_CAPACITY_OVERFLOW;
      else nblk = count;
    }
    // work items of item_blocks groups of group_x horizontally adjacent blocks 
    const int ib = P.item_blocks[pl.level], gx = P.group_x[pl.level];
    const int nitem = nblk > 0 ? (block_groups(pl.nbx, pl.nby, gx) + ib - 1) / ib : 0;
    const int c0 = (pl.status == -1 && pl.level == 0) ? nitem : 0;
    const int c1 = (pl.status == -1 && pl.level == 1) ? nitem : 0;
    const int incl0 = wave_incl_scan(c0);
    const int incl1 = wave_incl_scan(c1);
    if (i < n) {
      const int g = fr.box_off + i;
      pl.off = off;
      pl.nblk = nblk;
      pl.ioff = pl.level == 0 ? carry0 + incl0 - c0 : carry1 + incl1 - c1;
      pl.frame = f;
      ws.plan[g] = pl;
      ws.clip[g] = cl;
      ws.litem_end[g] = carry0 + incl0;
      ws.litem_end[n_total + g] = carry1 + incl1;
    }
    carry += __builtin_amdgcn_readlane(incl, 63);
    carry0 += __builtin_amdgcn_readlane(incl0, 63);
    carry1 += __builtin_amdgcn_readlane(incl1, 63);
  }
  if (lane == 0) {
    int32_t* fc = ws.fcount + f * FC_N;
    fc[FC_NUMBERED] = carry;
    fc[FC_FAR_ITEMS] = carry0;
    fc[FC_CLOSE_ITEMS] = carry1;
  }
}

// ---------------------------------------------------------------------------------
// per-block steps
// ---------------------------------------------------------------------------------
// The first of the n running ends that passes q (the last one otherwise): one ballot per
// 64, the loads of 256 issued together. Above 256 ends, 64 of them that are `step` apart
// first say between which two to look (the ends do not decrease): an item's search of 20000
// boxes takes three loads in turn, where one through all of them took 79 and a 1080p frame of
// that many small boxes 3.6 ms instead of 2.8 (10000: 1.47 instead of 1.18 ms).
__device__ __forceinline__ int find_box(const int32_t* __restrict__ end, int n, int q, int lane) {
  int first = 0, left = n;                      // the answer is among ends first .. first + left - 1
  while (left > 256) {
    const int step = (left + 63) >> 6;
    const int at = min(step * (lane + 1), left) - 1;
    const uint64_t m = __ballot(end[first + at] > q);
    if (!m) return n - 1;
    const int k = __ffsll((unsigned long long)m) - 1;
    first += step * k;
    left = min(step, left - step * k);
  }
  int e[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = 64 * u + lane;
    e[u] = 0x7FFFFFFF;
    if (64 * u < left && i < left) e[u] = end[first + i];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint64_t m = __ballot(e[u] > q);
    if (m) return min(first + 64 * u + __ffsll((unsigned long long)m) - 1, n - 1);
  }
  return n - 1;
}

// Work item q of frame f's level: its box, found on the running item ends of the plan, and
// the box's block geometry. The plan holds one record per box and none per item: a frame's
// plan is one wave's work, and writing thousands of item records from it took most of a
// many-box frame's time (3840 x 2160 with 200 boxes: 155 us of census and plan).
__device__ __forceinline__ ItemRec find_item(const MatchParamsDev& P, const FrameDev& fr, int n_total,
                                             const MatchWs& ws, int level, int q, int lane) {
  const int k = find_box(ws.litem_end + (size_t)level * n_total + fr.box_off, fr.n_boxes, q, lane);
  const BoxPlan pl = ws.plan[fr.box_off + k];
  ItemRec r;
  r.k = k;
  r.sub = -1;
  r.first = uniform((q - pl.ioff) * P.item_blocks[level]);
  r.nblk = uniform(pl.nblk); r.ngrp = uniform(block_groups(pl.nbx, pl.nby, P.group_x[level])); r.off = uniform(pl.off);
  r.nbx = uniform(pl.nbx); r.bw = uniform(pl.bw); r.bh = uniform(pl.bh);
  r.ox = uniform(pl.ox); r.oy = uniform(pl.oy);
  r.lx0 = uniform(pl.lx0); r.ly0 = uniform(pl.ly0); r.lw = uniform(pl.lw); r.lh = uniform(pl.lh);
  return r;
}

struct BlockGeom {
  int nx, ny;
  int s;
  int tiled;
  int cx, lx0, lw;   // TILED: first column cx; GRID: lx0, lw
  int cy, ly0, lh;
};

__device__ __forceinline__ int geom_col(const BlockGeom& g, int i) {
  return g.tiled ? g.cx + i : g.lx0 + (2 * i + 1) * g.lw / (2 * g.nx);
}
__device__ __forceinline__ int geom_row(const BlockGeom& g, int j) {
  return g.tiled ? g.cy + j : g.ly0 + (2 * j + 1) * g.lh / (2 * g.ny);
}

// Occlusion-aware sampling (Sec. 4.3.5): bit j*nx+i is set iff point (i, j) lies in no
// box of the frame that overlaps box k and has a larger bottom y. Lanes scan the boxes
// 64 at a time; the few occluders found are then tested against one point per lane.
__device__ __forceinline__ uint64_t block_mask(const MatchWs& ws, int box_off, int n, int k,
                                               const BlockGeom& g, int lane) {
  const BoxClip ck = ws.clip[box_off + k];
  const int s = g.s;
  const int npts = g.nx * g.ny;
  const int pi = lane % g.nx, pj = min(lane / g.nx, g.ny - 1);
  const int fx = s * geom_col(g, pi), fy = s * geom_row(g, pj);
  const int bx0 = s * geom_col(g, 0), bx1 = s * geom_col(g, g.nx - 1);
  const int by0 = s * geom_row(g, 0), by1 = s * geom_row(g, g.ny - 1);
  bool hidden = false;
  for (int jb = 0; jb < n; jb += 64) {
    const int o = jb + lane;
    const BoxClip co = o < n ? ws.clip[box_off + o] : BoxClip{0, 0, 0, 0};
    const bool occ = o < n && o != k && ck.cx0 < co.cx1 && co.cx0 < ck.cx1 && ck.cy0 < co.cy1 &&
                     co.cy0 < ck.cy1 && co.cy1 > ck.cy1 && co.cx0 <= bx1 && co.cx1 > bx0 &&
                     co.cy0 <= by1 && co.cy1 > by0;
    uint64_t m = __ballot(occ);
    while (m) {
      // the occluder's box, read from the lane that loaded it
      const int src = __ffsll((unsigned long long)m) - 1;
      m &= m - 1;
      const int x0 = __builtin_amdgcn_readlane(co.cx0, src), x1 = __builtin_amdgcn_readlane(co.cx1, src);
      const int y0 = __builtin_amdgcn_readlane(co.cy0, src), y1 = __builtin_amdgcn_readlane(co.cy1, src);
      hidden |= fx >= x0 && fx < x1 && fy >= y0 && fy < y1;
    }
  }
  return __ballot(lane < npts && !hidden);
}

__device__ __forceinline__ bool block_eligible(const MatchParamsDev& P, uint64_t mask, int npts) {
  const int nm = __popcll(mask);
  return nm > 0 && 100 * nm >= P.min_point_pct * npts;
}

// parabola through (d_f - 1, a), (d_f, c), (d_f + 1, b) (sub-pixel equation, in d = -dx);
// at either end of the range the integer disparity is kept
__device__ __forceinline__ float subpixel(int d_f, int best, int nd, int a, int c, int b) {
  if (best > 0 && best < nd - 1) {
    const int num = a - b;
    const int den = 2 * (a + b - 2 * c);
    const float offs = (float)num / (float)den;
    return (float)d_f + offs;
  }
  return (float)d_f;
}

struct BlockCtx {
  int f;            // frame index
  int level;
  int k;            // box index within the frame
  int kg;           // box index over the call
  int b;            // block number within the frame
  int slot;         // block storage index over the call
  int u, v;
  BoxPlan pl;
  BlockGeom g;
};

// block `local` (0-based, row-major over the box's block grid) of box k of frame f, at
// column u and row v of the grid
__device__ __forceinline__ BlockCtx block_ctx(const MatchParamsDev& P, const FrameDev& fr, int f,
                                              int k, const BoxPlan& pl, int local, int u, int v,
                                              int level) {
  BlockCtx c;
  c.f = f;
  c.level = level;
  c.k = k;
  c.kg = fr.box_off + k;
  c.pl = pl;
  c.b = pl.off + local;
  c.slot = f * P.cap_blocks + c.b;
  c.v = v;
  c.u = u;
  const LevelDev& lv = fr.lv[level];
  c.g.nx = pl.bw; c.g.ny = pl.bh; c.g.s = lv.scale;
  c.g.tiled = P.path[level].mode == OCSR_MODE_TILED;
  c.g.cx = pl.ox + c.u * pl.bw; c.g.lx0 = pl.lx0; c.g.lw = pl.lw;
  c.g.cy = pl.oy + c.v * pl.bh; c.g.ly0 = pl.ly0; c.g.lh = pl.lh;
  return c;
}
__device__ __forceinline__ BlockCtx block_ctx(const MatchParamsDev& P, const FrameDev& fr, int f,
                                              int k, const BoxPlan& pl, int local, int level) {
  const int v = local / pl.nbx;
  return block_ctx(P, fr, f, k, pl, local, local - v * pl.nbx, v, level);
}

// Stores the block's result (lane 0 of the wave).
__device__ __forceinline__ void write_block(const MatchWs& ws, const DebugDev& dbg,
                                            const BlockCtx& c, const PathDev& ph, uint64_t mask,
                                            bool eligible, int d_f, int d_b, int lr_ok,
                                            float d_sub, int valid, int lane, int dy_f = 0,
                                            int dy_b = 0) {
  if (lane == 0) {
    ws.blk_val[c.slot] = (float)c.g.s * d_sub;   // d_full = s * d (Sec. 4.1)
    ws.blk_flag[c.slot] = (uint8_t)((eligible ? 1 : 0) | (valid ? 2 : 0));
    if (dbg.blocks && c.b < dbg.cap_blocks) {
      ocsr_block_record rec;
      rec.box = c.k; rec.level_scale = c.g.s; rec.u = c.u; rec.v = c.v;
      rec.px0 = geom_col(c.g, 0); rec.py0 = geom_row(c.g, 0); rec.nx = c.g.nx; rec.ny = c.g.ny;
      rec.mask = mask; rec.eligible = eligible; rec.d_f = d_f; rec.d_b = d_b;
      rec.lr_ok = lr_ok; rec.d_sub = d_sub; rec.valid = valid;
      rec.dlo = ph.dlo; rec.nd = ph.nd;
      rec.dy_f = dy_f; rec.dy_b = dy_b;
      dbg.blocks[c.b] = rec;
    }
  }
}

// ---------------------------------------------------------------------------------
// TILED block, register-blocked. One wave per block of at most NX x ROWS points.
// Lane = (row j, candidate group g); group g owns CPL consecutive candidates. The
// block's template rows and its search strip (nd + nx - 1 words per row) are staged
// in LDS with coalesced loads; each lane then holds its row's NX template words and
// NX + CPL - 1 strip words in registers and forms NX * CPL costs from them
// (2 x v_xor_b32 + 2 x v_bcnt_u32_b32 each). Row sums are combined with DPP.
// ---------------------------------------------------------------------------------
// popcount of a 64-bit word added to acc as two v_bcnt_u32_b32 (each adds its popcount
// to its second operand). Written as instructions so that the compiler cannot regroup a
// chain of these sums into popcounts of zero plus v_add3_u32 adds, which costs a fifth
// instruction per term.
__device__ __forceinline__ uint32_t popc64_acc(uint64_t x, uint32_t acc) {
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"((uint32_t)x));
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"((uint32_t)(x >> 32)));
  return acc;
}

// acc[c] = sum over the row's unmasked points i of popcount(t[i] ^ srow[i + c]).
// col_all / col_any (wave-uniform): the block columns whose point is unmasked in every
// row / in some row. Columns masked in every row (occluded, or past the block's width)
// are skipped. When every other column is unmasked in every row, a cost is 4 ops;
// otherwise each difference is ANDed with the lane's own mask bit (6 ops).
template <int NX, int CPL>
__device__ __forceinline__ void row_costs(const uint64_t (&t)[NX], const uint64_t* __restrict__ srow,
                                          uint32_t rowmask, uint32_t col_all, uint32_t col_any,
                                          uint32_t (&acc)[CPL]) {
  uint64_t w[NX + CPL - 1];
#pragma unroll
  for (int m = 0; m < NX + CPL - 1; ++m) w[m] = srow[m];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = 0;
  if (col_all == col_any) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      if (col_all & (1u << i)) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = popc64_acc(t[i] ^ w[i + c], acc[c]);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      if (col_any & (1u << i)) {
        const uint64_t keep = ((rowmask >> i) & 1u) ? ~0ull : 0ull;
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = popc64_acc((t[i] ^ w[i + c]) & keep, acc[c]);
      }
    }
  }
}

template <int ROWS>
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
  // lanes j = lane % ROWS of one group: quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
  if (ROWS == 8) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);
  return v;
}

// S[jj * SW + m] = row jj's word at x_first + m of the level image (0 outside the
// image, past the block's ny rows or past sw words), for ROWS x SW entries. All loads
// of a lane are issued before the first is waited for; an entry with no word reads
// the block's first row at column 0 instead and is zeroed.
template <int ROWS, int SW>
__device__ __forceinline__ void stage_strip(uint64_t* __restrict__ S, const uint64_t* __restrict__ rows,
                                            int pitch, int x_first, int ny, int sw, int W, int lane) {
  if constexpr ((SW & (SW - 1)) == 0) {
    // power-of-two rows: word idx = lane + 64 k of the ROWS x SW strip, row and column
    // by shift and mask
    constexpr int N = ROWS * SW, IT = (N + 63) / 64;
    uint64_t w[IT];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int idx = lane + 64 * k;
      const int jj = idx / SW, m = idx % SW, x = x_first + m;
      const bool ok = idx < N && jj < ny && m < sw && x >= 0 && x < W;
      w[k] = rows[ok ? (size_t)jj * pitch + x : 0];
      w[k] = ok ? w[k] : 0ull;
    }
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int idx = lane + 64 * k;
      if (idx < N) S[idx] = w[k];
    }
  } else {
    // row by row in chunks of 64 words: the row is a constant and the column the lane,
    // so no per-lane division (whose results the compiler would keep live in registers
    // across the whole work-item loop)
    constexpr int CH = (SW + 63) / 64;
    uint64_t w[ROWS][CH];
#pragma unroll
    for (int jj = 0; jj < ROWS; ++jj)
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int m = 64 * c + lane, x = x_first + m;
        const bool ok = jj < ny && m < sw && x >= 0 && x < W;
        w[jj][c] = rows[ok ? (size_t)jj * pitch + x : 0];
        w[jj][c] = ok ? w[jj][c] : 0ull;
      }
#pragma unroll
    for (int jj = 0; jj < ROWS; ++jj)
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (64 * c + lane < SW) S[jj * SW + 64 * c + lane] = w[jj][c];
  }
}

template <int ROWS, int NX, int CPL, int PASSES = 1>
struct Tiled {
  static constexpr int G = 64 / ROWS;
  static constexpr int NC = G * CPL * PASSES;  // candidates one wave covers
  static constexpr int SW = NC + NX - 1;       // strip words per row
  static constexpr size_t kLdsBytes = sizeof(uint64_t) * (ROWS * SW + ROWS * NX) +
                                      sizeof(uint32_t) * 2 * NC;
  static_assert(ROWS == 4 || ROWS == 8, "rows");
};

template <int ROWS, int NX, int CPL, int PASSES = 1>
__device__ __forceinline__ void match_block_tiled(const MatchParamsDev& P, const FrameDev& fr,
                                                  const MatchWs& ws, const DebugDev& dbg,
                                                  const BlockCtx& c, int lane, void* lds) {
  using TT = Tiled<ROWS, NX, CPL, PASSES>;
  constexpr int PC = TT::G * CPL;              // candidates of one pass
  constexpr int SW = TT::SW, NC = TT::NC;
  uint64_t* S = (uint64_t*)lds;
  uint64_t* T = S + ROWS * SW;
  uint32_t* costf = (uint32_t*)(T + ROWS * NX);
  uint32_t* costb = costf + NC;
  const int j = lane % ROWS, grp = lane / ROWS;
  const LevelDev& lv = fr.lv[c.level];
  const PathDev& ph = P.path[c.level];
  const int nd = ph.nd, dlo = ph.dlo, dhi = dlo + nd - 1;

  const int nx = c.g.nx, ny = c.g.ny;
  const int X0 = c.g.cx, Y0 = c.g.cy;
  const uint64_t* __restrict__ Lb = lv.L + (size_t)Y0 * lv.pitch;
  const uint64_t* __restrict__ Rb = lv.R + (size_t)Y0 * lv.pitch;
  const int sw = nd + nx - 1;
  // forward: template CL(X0 + i, Y0 + j); strip CR(X0 - dhi + m, Y0 + j). Issued before
  // the occluder scan so that both sets of loads are in flight together.
  stage_strip<ROWS, SW>(S, Rb, lv.pitch, X0 - dhi, ny, sw, lv.W, lane);
  stage_strip<ROWS, NX>(T, Lb, lv.pitch, X0, ny, nx, lv.W, lane);
  const uint64_t mask = block_mask(ws, fr.box_off, fr.n_boxes, c.k, c.g, lane);
  const bool eligible = block_eligible(P, mask, nx * ny);
  wave_sync();
  if (!eligible) {
    write_block(ws, dbg, c, ph, mask, false, dlo, dlo, 0, (float)dlo, 0, lane);
    wave_sync();
    return;
  }
  const uint32_t rowmask = j < ny ? (uint32_t)((mask >> (j * nx)) & ((1u << nx) - 1u)) : 0u;
  // columns unmasked in every row / in some row (the mask is wave-uniform)
  uint32_t col_all = (1u << nx) - 1u, col_any = 0;
  for (int jj = 0; jj < ny; ++jj) {
    const uint32_t r = (uint32_t)((mask >> (jj * nx)) & ((1u << nx) - 1u));
    col_all &= r;
    col_any |= r;
  }
  uint64_t t[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) t[i] = T[j * NX + i];
  uint32_t acc[CPL];
  uint32_t key = 0xFFFFFFFFu;
  // strip entry e + i (e = ps*PC + grp*CPL + c) holds CR(X0 + i - d) for d = dhi - e;
  // the candidates are covered in PASSES passes of PC
#pragma unroll 1
  for (int ps = 0; ps < PASSES; ++ps) {
    if (j < ny) row_costs<NX, CPL>(t, S + j * SW + ps * PC + grp * CPL, rowmask, col_all, col_any, acc);
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc)
      if (j >= ny) acc[cc] = 0;
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const uint32_t tot = row_sum<ROWS>(acc[cc]);
      const int e = ps * PC + grp * CPL + cc;
      if (e < nd) {
        const int kc = nd - 1 - e;
        key = min(key, (tot << 16) | (uint32_t)kc);
        if (j == 0) costf[kc] = tot;
      }
    }
  }
  key = wave_min_u32(key, ROWS);
  const int best = (int)(key & 0xFFFFu);
  const int d_f = dlo + best;
  // backward template CR(X0 - d_f + i, Y0 + j) sits in the forward strip at dhi - d_f + i
#pragma unroll
  for (int i = 0; i < NX; ++i) t[i] = S[j * SW + (dhi - d_f) + i];
  wave_sync();
  const int ca = (int)costf[max(best - 1, 0)];
  const int cb = (int)costf[min(best + 1, nd - 1)];
  const float d_sub = subpixel(d_f, best, nd, ca, (int)(key >> 16), cb);
  // backward strip: CL(X0 - d_f + dlo + m, Y0 + j)
  stage_strip<ROWS, SW>(S, Lb, lv.pitch, X0 - d_f + dlo, ny, sw, lv.W, lane);
  wave_sync();
  uint32_t bkey = 0xFFFFFFFFu;
#pragma unroll 1
  for (int ps = 0; ps < PASSES; ++ps) {
    if (j < ny) row_costs<NX, CPL>(t, S + j * SW + ps * PC + grp * CPL, rowmask, col_all, col_any, acc);
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc)
      if (j >= ny) acc[cc] = 0;
#pragma unroll
    for (int cc = 0; cc < CPL; ++cc) {
      const uint32_t tot = row_sum<ROWS>(acc[cc]);
      const int kc = ps * PC + grp * CPL + cc;   // candidate dlo + kc
      if (kc < nd) {
        bkey = min(bkey, (tot << 16) | (uint32_t)kc);
        if (j == 0) costb[kc] = tot;
      }
    }
  }
  bkey = wave_min_u32(bkey, ROWS);
  const int d_b = dlo + (int)(bkey & 0xFFFFu);
  const int lr_ok = abs(d_b - d_f) <= P.lr_tol;
  if (c.b < dbg.cap_blocks && (dbg.cost_fwd || dbg.cost_bwd)) {
    wave_sync();
    for (int kc = lane; kc < nd && kc < dbg.cap_nd; kc += 64) {
      if (dbg.cost_fwd) dbg.cost_fwd[(size_t)c.b * dbg.cap_nd + kc] = (uint16_t)costf[kc];
      if (dbg.cost_bwd) dbg.cost_bwd[(size_t)c.b * dbg.cap_nd + kc] = (uint16_t)costb[kc];
    }
  }
  write_block(ws, dbg, c, ph, mask, true, d_f, d_b, lr_ok, d_sub, lr_ok, lane);
  wave_sync();
}

// Whole-wave minimum of v (every lane gets it): DPP within rows of 16, then row
// broadcasts (lane 15 into the next row, lane 31 into rows 2 and 3), then lane 63.
__device__ __forceinline__ uint32_t wave_min_dpp(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Minimum over each row of 16 lanes (every lane of the row gets it).
__device__ __forceinline__ uint32_t row16_min_dpp(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));
  return v;
}

// Whether point (fx, fy) lies in one of the rectangles held by the lanes of m (each lane
// o holds the clipped box co).
__device__ __forceinline__ bool in_lane_rects(uint64_t m, const BoxClip& co, int fx, int fy) {
  bool hidden = false;
  while (m) {
    const int src = __ffsll((unsigned long long)m) - 1;
    m &= m - 1;
    const int x0 = __builtin_amdgcn_readlane(co.cx0, src), x1 = __builtin_amdgcn_readlane(co.cx1, src);
    const int y0 = __builtin_amdgcn_readlane(co.cy0, src), y1 = __builtin_amdgcn_readlane(co.cy1, src);
    hidden |= fx >= x0 && fx < x1 && fy >= y0 && fy < y1;
  }
  return hidden;
}

// The boxes that may hide points of box k, for all blocks of one work item of a frame of
// at most 64 boxes (in_lanes): lane o holds box o's clipped rectangle, and bit o of `cand` is
// set iff box o overlaps box k and has the larger bottom y, the part of the occlusion
// test (Sec. 4.3.5) that does not depend on the block.
struct OccLanes {
  BoxClip co;
  uint64_t cand;
  bool in_lanes;
};
// The frame's part, which does not depend on k (so its load need not wait for an item
// record): lane o holds box o's clipped rectangle.
__device__ __forceinline__ OccLanes frame_lanes(const MatchWs& ws, int box_off, int n, int lane) {
  OccLanes oc{BoxClip{0, 0, 0, 0}, 0ull, n <= 64};
  if (oc.in_lanes && lane < n) oc.co = ws.clip[box_off + lane];
  return oc;
}
// Box k's candidates (box k's own rectangle from lane k).
__device__ __forceinline__ void box_candidates(OccLanes& oc, int n, int k, int lane) {
  if (!oc.in_lanes) return;
  const BoxClip co = oc.co;
  const BoxClip ck{__builtin_amdgcn_readlane(co.cx0, k), __builtin_amdgcn_readlane(co.cy0, k),
                   __builtin_amdgcn_readlane(co.cx1, k), __builtin_amdgcn_readlane(co.cy1, k)};
  oc.cand = __ballot(lane < n && lane != k && ck.cx0 < co.cx1 && co.cx0 < ck.cx1 &&
                     ck.cy0 < co.cy1 && co.cy0 < ck.cy1 && co.cy1 > ck.cy1);
}
// ---------------------------------------------------------------------------------
// Any block of up to 64 points on any point grid (TILED, or the single GRID block of
// the paper's far path, Sec. 4.3.4 "Far Objects"), up to 256 candidates: one wave per
// block. The kept points are listed in LDS (template word, offset and column); lane l takes
// candidate l (and l + 64, ..), and with at most 32 (16) candidates the wave's halves
// (quarters) share the points out. Each step loads eight points' candidate words before
// it uses any: a GRID level has few blocks, one per far box, and a wave that waits for
// each of 64 points in turn was all its time (48 boxes of a
// 1080p frame, both levels: 53 us, now 18).
// Reads of the level images are checked against [0, W); point rows lie inside the level
// box.
// ---------------------------------------------------------------------------------
struct GenericLds {
  uint32_t costf[256], costb[256];
  uint64_t tmpl[64 + 8];      // the listed points' template words; 0 past the end
  int64_t row[64 + 8];        // their row's first word
  int32_t x[64 + 8];          // their column (forward) or match column (backward)
};
constexpr size_t kGenericLdsBytes = sizeof(GenericLds);

// acc[r]: the cost of candidate l + 64 r over the n listed points, l = lane mod (64 / ng).
// Candidate kc of a point reads column x + step (dlo + kc) of img.
__device__ __forceinline__ void generic_costs(const GenericLds& sm, const uint64_t* __restrict__ img, int W,
                                              int n, int dlo, int nd, int step, int ng, int lane,
                                              uint32_t (&acc)[4]) {
  constexpr int B = 8;
  const int per = 64 / ng, l = lane & (per - 1), grp = lane / per;
  acc[0] = acc[1] = acc[2] = acc[3] = 0;
  for (int i0 = 0; i0 < n; i0 += B * ng) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (64 * r >= nd) break;   // wave-uniform
      const int kc = l + 64 * r;
      const int dx = step * (dlo + kc);
      uint64_t w[B], t[B];
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const int i = min(i0 + j * ng + grp, n);      // entry n: a word that differs from none
        const int xc = sm.x[i] + dx;
        const bool ok = kc < nd && i < n && xc >= 0 && xc < W;
        t[j] = sm.tmpl[i];
        w[j] = img[ok ? sm.row[i] + xc : 0];
        w[j] = ok ? w[j] : 0ull;
      }
#pragma unroll
      for (int j = 0; j < B; ++j) acc[r] = popc64_acc(t[j] ^ w[j], acc[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (ng >= 2) acc[r] += (uint32_t)__shfl_xor((int)acc[r], 32, 64);
    if (ng == 4) acc[r] += (uint32_t)__shfl_xor((int)acc[r], 16, 64);
  }
}

// The same over at most kFewPoints points, which are not listed: lane t holds point t's template
// word (0 where it is not kept), row and column. The list would have every candidate word wait
// for the template words, a load's latency per direction that one round of points does not win
// back: 1080p frames of single-point blocks 20 to 25 us with the list, 18 to 23 without.
constexpr int kFewPoints = 4;
__device__ __forceinline__ void few_point_costs(const uint64_t* __restrict__ img, int W, uint64_t mask,
                                                uint64_t word, int64_t row, int x, int dlo, int nd,
                                                int step, int lane, uint32_t (&acc)[4]) {
  auto lane_word = [](uint64_t v, int src) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), src) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)v, src);
  };
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    acc[r] = 0;
    if (64 * r >= nd) continue;                 // wave-uniform
    const int kc = lane + 64 * r;
    uint64_t w[kFewPoints], m = mask;
    int src[kFewPoints];
#pragma unroll
    for (int j = 0; j < kFewPoints; ++j) {
      src[j] = m ? __ffsll((unsigned long long)m) - 1 : -1;
      m &= m - 1;
      w[j] = 0;
      if (src[j] >= 0) {
        const int xc = __builtin_amdgcn_readlane(x, src[j]) + step * (dlo + kc);
        const bool ok = kc < nd && xc >= 0 && xc < W;
        w[j] = img[ok ? (int64_t)lane_word((uint64_t)row, src[j]) + xc : 0];
        w[j] = ok ? w[j] : 0ull;
      }
    }
#pragma unroll
    for (int j = 0; j < kFewPoints; ++j)
      if (src[j] >= 0) acc[r] = popc64_acc(lane_word(word, src[j]) ^ w[j], acc[r]);
  }
}

__device__ __forceinline__ void match_block_generic(const MatchParamsDev& P, const FrameDev& fr,
                                                    const MatchWs& ws, const DebugDev& dbg,
                                                    const BlockCtx& c, int lane, void* lds) {
  GenericLds& sm = *(GenericLds*)lds;
  const LevelDev& lv = fr.lv[c.level];
  const PathDev& ph = P.path[c.level];
  const int nd = ph.nd, dlo = ph.dlo, W = lv.W;
  // lane t's point (t mod nx, t / nx); its word is loaded while the occluders are
  const bool point = lane < c.g.nx * c.g.ny;
  const int pj = lane / c.g.nx, pi = lane - pj * c.g.nx;
  const int px = point ? geom_col(c.g, pi) : 0;
  const int64_t prow = point ? (int64_t)geom_row(c.g, pj) * lv.pitch : 0;
  uint64_t word = ld_word(lv.L + prow, px, W);
  const uint64_t mask = block_mask(ws, fr.box_off, fr.n_boxes, c.k, c.g, lane);
  const bool eligible = block_eligible(P, mask, c.g.nx * c.g.ny);
  if (!eligible) {
    write_block(ws, dbg, c, ph, mask, false, dlo, dlo, 0, (float)dlo, 0, lane);
    wave_sync();
    return;
  }
  // the kept points' list: each at its rank in the mask
  const int n = (int)__popcll(mask);
  const bool few = n <= kFewPoints;
  const bool kept = (mask >> lane) & 1ull;
  const int at = (int)__popcll(mask & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
  if (!few) {
    if (kept) {
      sm.tmpl[at] = word;
      sm.row[at] = prow;
      sm.x[at] = px;
    }
    if (lane == 0) {
      sm.tmpl[n] = 0;
      sm.row[n] = 0;
      sm.x[n] = 0;
    }
    wave_sync();
  }
  const int ng = few ? 1 : nd <= 16 ? 4 : nd <= 32 ? 2 : 1;
  const bool lead = lane < 64 / ng;             // one lane per candidate
  uint32_t acc[4];
  // forward: CL(x) against CR(x - d)
  if (few) few_point_costs(lv.R, W, mask, word, prow, px, dlo, nd, -1, lane, acc);
  else generic_costs(sm, lv.R, W, n, dlo, nd, -1, ng, lane, acc);
  uint32_t key = 0xFFFFFFFFu;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int kc = lane + 64 * r;
    if (lead && kc < nd) {
      key = min(key, (acc[r] << 16) | (uint32_t)kc);
      sm.costf[kc] = acc[r];
    }
  }
  key = wave_min_dpp(key);
  const int best = (int)(key & 0xFFFFu);
  const int d_f = dlo + best;
  wave_sync();
  const int ca = (int)sm.costf[max(best - 1, 0)];
  const int cb = (int)sm.costf[min(best + 1, nd - 1)];
  const float d_sub = subpixel(d_f, best, nd, ca, (int)(key >> 16), cb);
  // backward: CR(x - d_f) against CL(x - d_f + d')
  if (kept) word = ld_word(lv.R + prow, px - d_f, W);
  if (few) {
    few_point_costs(lv.L, W, mask, word, prow, px - d_f, dlo, nd, 1, lane, acc);
  } else {
    if (kept) {
      sm.tmpl[at] = word;
      sm.x[at] = px - d_f;
    }
    wave_sync();
    generic_costs(sm, lv.L, W, n, dlo, nd, 1, ng, lane, acc);
  }
  uint32_t bkey = 0xFFFFFFFFu;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int kc = lane + 64 * r;
    if (lead && kc < nd) {
      bkey = min(bkey, (acc[r] << 16) | (uint32_t)kc);
      sm.costb[kc] = acc[r];
    }
  }
  bkey = wave_min_dpp(bkey);
  const int d_b = dlo + (int)(bkey & 0xFFFFu);
  const int lr_ok = abs(d_b - d_f) <= P.lr_tol;
  if (c.b < dbg.cap_blocks && (dbg.cost_fwd || dbg.cost_bwd)) {
    wave_sync();
    for (int kc = lane; kc < nd && kc < dbg.cap_nd; kc += 64) {
      if (dbg.cost_fwd) dbg.cost_fwd[(size_t)c.b * dbg.cap_nd + kc] = (uint16_t)sm.costf[kc];
      if (dbg.cost_bwd) dbg.cost_bwd[(size_t)c.b * dbg.cap_nd + kc] = (uint16_t)sm.costb[kc];
    }
  }
  write_block(ws, dbg, c, ph, mask, true, d_f, d_b, lr_ok, d_sub, lr_ok, lane);
  wave_sync();
}

// Work item of frame f at `level`: wave w of the workgroup runs blocks
// r.first + w + 4 j of the box that exist.
__device__ __forceinline__ BoxPlan item_plan(const ItemRec& r, int f, int level) {
  BoxPlan pl = {};
  pl.status = -1;
  pl.level = level;
  pl.lx0 = r.lx0; pl.ly0 = r.ly0; pl.lw = r.lw; pl.lh = r.lh;
  pl.nbx = r.nbx; pl.bw = r.bw; pl.bh = r.bh; pl.ox = r.ox; pl.oy = r.oy;
  pl.off = r.off; pl.nblk = r.nblk; pl.frame = f;
  return pl;
}
template <class RunBlock>
__device__ __forceinline__ void run_item_rec(const MatchParamsDev& P, const FrameDev& fr, int f,
                                             int level, const ItemRec& r, int wave, RunBlock run) {
  const BoxPlan pl = item_plan(r, f, level);
  // the wave's blocks step by kItemWaves along the grid's rows: one division per item
  int local = r.first + wave;
  int v = local / pl.nbx, u = local - v * pl.nbx;
  for (int j = wave; j < P.item_blocks[level]; j += kItemWaves) {
    if (local < r.nblk) run(block_ctx(P, fr, f, r.k, pl, local, u, v, level));
    local += kItemWaves;
    u += kItemWaves;
    while (u >= pl.nbx) {
      u -= pl.nbx;
      ++v;
    }
  }
}

// log2 of the units that an item of kItemWaves groups is dealt in: one, or kItemWaves where the
// call's n items hold at most share_groups groups (0: never).
__device__ __forceinline__ int share_items(int n, int share_groups) {
  static_assert(kItemWaves == 4, "units of a quarter");
  return n <= share_groups / kItemWaves ? (share_groups > 0 ? 2 : 0) : 0;
}

// Loop of a workgroup over the work items of one level of every frame (frames in
// order, each frame's items in box order), dealt XCD by XCD (xcd_deal). Item numbers
// come from the workgroup index, so the loop is uniform across the workgroup and needs
// no shared counter. body(f, q, sub) gets the frame, the item number within the frame's
// level and -1; or, where the items hold at most share_groups groups (kItemWaves each), the
// items' groups are dealt one by one and sub is the group's number within its item.
template <class Body>
__device__ __forceinline__ void level_items(const FramesDev& FR, const MatchWs& ws, int level,
                                            int share_groups, Body body) {
  const int lane = threadIdx.x & 63;
  const int cnt = lane < FR.n ? ws.fcount[lane * FC_N + (level == 0 ? FC_FAR_ITEMS : FC_CLOSE_ITEMS)] : 0;
  const int incl = wave_incl_scan(cnt);
  const int total = __builtin_amdgcn_readlane(incl, 63);
  const int sh = share_items(total, share_groups);
  const Deal dl = xcd_deal(total << sh);
  for (int i = dl.first; i < dl.end; i += dl.step) {
    const int q = i >> sh;
    const uint64_t m = __ballot(lane < FR.n && incl > q);
    const int f = __ffsll((unsigned long long)m) - 1;
    body(f, q - __builtin_amdgcn_readlane(incl - cnt, f), sh ? i & (kItemWaves - 1) : -1);
  }
}

// ---------------------------------------------------------------------------------
// aggregation: one workgroup (256 threads) per box
// ---------------------------------------------------------------------------------
struct AggLds {
  float vals[kAggMax];    // the box's valid values (boxes of at most kAggMax blocks)
  int32_t hist[1024];     // value histogram of the trimmed median; per-wave digit counts
                          // of the global radix sort ([kItemWaves][256])
  uint32_t lo[1024], hi[1024];   // smallest and largest value (bit patterns) of the bins
                          // beside an empty one (segment median)
  unsigned long long run; // longest run: length << 32 | ~(its number)
  float list[2][64];      // values of the bins holding the two middle ranks
  int32_t scratch[272];   // radix bins [0, 256), then scalars
  int32_t n_valid, n_eligible, seg_start, seg_len;
  uint32_t vmin, vmax;    // bit patterns of the smallest and largest valid value
  int32_t bin[2], rank[2], count[2];
  uint32_t pick[2];
};

__device__ __forceinline__ float median_sorted(const float* v, int m) {
  if (m & 1) return v[(m - 1) / 2];
  return (v[m / 2 - 1] + v[m / 2]) * 0.5f;
}

// k-th smallest (0-based) of the n non-negative floats in vals (LDS or global memory):
// radix select on their bit patterns (monotone for non-negative floats), 8 bits per pass
__device__ __forceinline__ uint32_t radix_select(const float* vals, int n, int k, int32_t* sc) {
  const int tid = threadIdx.x;
  uint32_t prefix = 0, pmask = 0;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    sc[tid] = 0;   // 256 bins
    __syncthreads();
    for (int i = tid; i < n; i += 256) {
      const uint32_t u = __float_as_uint(vals[i]);
      if ((u & pmask) == prefix) atomicAdd(&sc[(u >> shift) & 255u], 1);
    }
    __syncthreads();
    if (tid < 64) {
      const int c0 = sc[4 * tid], c1 = sc[4 * tid + 1], c2 = sc[4 * tid + 2], c3 = sc[4 * tid + 3];
      const int sum = c0 + c1 + c2 + c3;
      const int incl = wave_incl_scan(sum);
      const int excl = incl - sum;
      if (k >= excl && k < incl) {   // exactly one lane
        int d = 4 * tid, kk = k - excl;
        if (kk >= c0) { kk -= c0; ++d;
          if (kk >= c1) { kk -= c1; ++d;
            if (kk >= c2) { kk -= c2; ++d; } } }
        sc[256] = d;
        sc[257] = kk;
      }
    }
    __syncthreads();
    prefix |= (uint32_t)sc[256] << shift;
    pmask |= 255u << shift;
    k = sc[257];
    __syncthreads();
  }
  return prefix;
}

// Ascending sort of the n non-negative floats at a (global memory) by their bit
// patterns: four stable counting passes of 8 bits, least significant first, between a
// and tmp (n floats); the sorted values end in a. One workgroup of 256 threads. A pass
// counts the digits, scans them to the start of each digit's range, then scatters 256
// values at a time in index order: a value's place is its digit's start, plus the
// values of that digit in earlier waves of the round, plus those of lower lanes of its
// own wave (found with eight ballots, one per digit bit). cnt: kItemWaves x 256 ints,
// base: 256 ints of LDS.
__device__ __forceinline__ void radix_sort_global(float* a, float* tmp, int n, int32_t* cnt,
                                                  int32_t* base) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 8 * pass;
    const float* src = (pass & 1) ? tmp : a;
    float* dst = (pass & 1) ? a : tmp;
    base[tid] = 0;
    for (int w = 0; w < kItemWaves; ++w) cnt[w * 256 + tid] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += 256) atomicAdd(&base[(__float_as_uint(src[i]) >> shift) & 255u], 1);
    __syncthreads();
    // exclusive scan of the 256 digit counts (thread t holds digit t)
    {
      const int c = base[tid];
      const int incl = wave_incl_scan(c);
      __syncthreads();
      if (lane == 63) cnt[wave] = incl;   // wave totals (cnt is all zero otherwise)
      __syncthreads();
      int excl = incl - c;
      for (int w = 0; w < wave; ++w) excl += cnt[w];
      __syncthreads();
      base[tid] = excl;
      if (tid < kItemWaves) cnt[tid] = 0;
      __syncthreads();
    }
    for (int c0 = 0; c0 < n; c0 += 256) {
      const int i = c0 + tid;
      const bool ok = i < n;
      const float v = ok ? src[i] : 0.0f;
      const uint32_t dg = (__float_as_uint(v) >> shift) & 255u;
      uint64_t same = __ballot(ok);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const uint64_t m = __ballot((dg >> b) & 1u);
        same &= ((dg >> b) & 1u) ? m : ~m;
      }
      const int before = (int)__popcll(same & below);
      if (ok && before == 0) cnt[wave * 256 + dg] = (int)__popcll(same);
      __syncthreads();
      if (ok) {
        int pos = base[dg] + before;
        for (int w = 0; w < wave; ++w) pos += cnt[w * 256 + dg];
        dst[pos] = v;
      }
      __syncthreads();
      int add = 0;
      for (int w = 0; w < kItemWaves; ++w) {
        add += cnt[w * 256 + tid];
        cnt[w * 256 + tid] = 0;
      }
      base[tid] += add;
      __syncthreads();
    }
  }
  // the last pass wrote into a; make its stores visible to the whole workgroup
  __threadfence_block();
  __syncthreads();
}

// Bin of v among 1024 equal-width bins over [vmin, vmin + 1024 / scale]: a monotone map,
// so every value of a lower bin is smaller than every value of a higher one.
__device__ __forceinline__ int value_bin(float v, float vmin, float scale) {
  return min((int)((v - vmin) * scale), 1023);
}

// Over the counts in sm.hist (1024 bins), the bins of ranks r1 and r2 (0-based; r2 only
// when want2) and the ranks within them, into sm.bin and sm.rank. All 256 threads; ends
// with a barrier.
__device__ __forceinline__ void find_rank_bins(AggLds& sm, int r1, int r2, bool want2) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // thread t owns bins 4t .. 4t + 3
  const int c0 = sm.hist[4 * tid], c1 = sm.hist[4 * tid + 1], c2 = sm.hist[4 * tid + 2],
            c3 = sm.hist[4 * tid + 3];
  const int sum = c0 + c1 + c2 + c3;
  const int incl = wave_incl_scan(sum);
  if (lane == 63) sm.scratch[256 + wave] = incl;
  __syncthreads();
  int excl = incl - sum;
  for (int v = 0; v < wave; ++v) excl += sm.scratch[256 + v];
  for (int j = 0; j < (want2 ? 2 : 1); ++j) {
    const int kj = j ? r2 : r1;
    if (kj >= excl && kj < excl + sum) {   // exactly one thread
      int b = 4 * tid, kk = kj - excl;
      if (kk >= c0) { kk -= c0; ++b;
        if (kk >= c1) { kk -= c1; ++b;
          if (kk >= c2) { kk -= c2; ++b; } } }
      sm.bin[j] = b;
      sm.rank[j] = kk;
    }
  }
  __syncthreads();
}

// The values whose key (key(v) < 1024, or -1 for none) is kb1 or kb2 gathered into the
// two lists (list 1 only when the keys differ), and the values of ranks sm.rank[0] and
// sm.rank[1] within their key picked by one wave into sm.pick. Every key count is at most
// 64. All 256 threads; ends with a barrier.
template <typename Key>
__device__ __forceinline__ void pick_in_lists(AggLds& sm, const float* vals, int n, Key key,
                                              int kb1, int kb2, bool want2) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < n; i += 256) {
    const float v = vals[i];
    const int b = key(v);
    if (b == kb1) sm.list[0][atomicAdd(&sm.count[0], 1)] = v;
    else if (b == kb2) sm.list[1][atomicAdd(&sm.count[1], 1)] = v;
  }
  __syncthreads();
  if (wave == 0) {
    for (int j = 0; j < (want2 ? 2 : 1); ++j) {
      const int li = (j == 1 && kb2 != kb1) ? 1 : 0;
      const int c = sm.count[li];
      const float* lst = sm.list[li];
      const float x = lane < c ? lst[lane] : 0.0f;
      int less = 0, eq = 0;
      for (int i = 0; i < c; ++i) {
        const float y = lst[i];
        less += y < x;
        eq += y == x;
      }
      // lanes holding equal values agree, so any of them may store
      if (lane < c && sm.rank[j] >= less && sm.rank[j] < less + eq) sm.pick[j] = __float_as_uint(x);
    }
  }
  __syncthreads();
}

// The k-th and (k + 1)-th smallest (0-based) of the n non-negative floats in vals (LDS
// or global memory; the second only when want2), as bit patterns. The values are binned
// by value (value_bin); a scan of the bin counts finds the bins of the two ranks and
// their ranks within them; one wave then ranks the few values of each such bin against
// each other. When a bin holds more than 64 values (a box's values crowd a few bins when
// a few outliers stretch the range), the values of the one or two bins are binned again
// over each bin's own span, 512 sub-bins each, and the same steps run on the sub-bins.
// A radix selection over all values handles a sub-bin of more than 64 values or a range
// too narrow to scale. vmin, vmax: the smallest and largest value. Every step is a
// monotone map of the value, so the order statistics are exact.
__device__ __forceinline__ void select_middle(AggLds& sm, const float* vals, int n, int k,
                                              bool want2, float vmin, float vmax, uint32_t* u1,
                                              uint32_t* u2) {
  const int tid = threadIdx.x;
  if (vmin == vmax) {
    *u1 = *u2 = __float_as_uint(vmin);
    return;
  }
  const float scale = 1024.0f / (vmax - vmin);
  if (scale < 1e30f) {
    for (int i = tid; i < n; i += 256) atomicAdd(&sm.hist[value_bin(vals[i], vmin, scale)], 1);
    if (tid == 0) { sm.count[0] = 0; sm.count[1] = 0; }
    __syncthreads();
    find_rank_bins(sm, k, k + 1, want2);
    const int b1 = sm.bin[0], b2 = want2 ? sm.bin[1] : b1;
    const int n1 = sm.hist[b1], n2 = sm.hist[b2];
    if (n1 <= 64 && n2 <= 64) {
      pick_in_lists(sm, vals, n, [&](float v) { return value_bin(v, vmin, scale); }, b1, b2, want2);
      *u1 = sm.pick[0];
      *u2 = want2 ? sm.pick[1] : sm.pick[0];
      return;
    }
    // second level: bin b1's values into sub-bins 0..511 and, when the second rank lies
    // in a later bin b2, bin b2's into 512..1023; ranks counted over the two bins together
    const int r1 = sm.rank[0], r2 = want2 ? (b2 == b1 ? sm.rank[1] : n1 + sm.rank[1]) : r1;
    auto sub = [&](float v) {
      const int b = value_bin(v, vmin, scale);
      if (b != b1 && b != b2) return -1;
      const int q = min(max((int)(((v - vmin) * scale - (float)b) * 512.0f), 0), 511);
      return b == b1 ? q : 512 + q;
    };
    __syncthreads();   // every thread has read the first level's counts
    for (int i = tid; i < 1024; i += 256) sm.hist[i] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += 256) {
      const int q = sub(vals[i]);
      if (q >= 0) atomicAdd(&sm.hist[q], 1);
    }
    __syncthreads();
    find_rank_bins(sm, r1, r2, want2);
    const int s1 = sm.bin[0], s2 = want2 ? sm.bin[1] : s1;
    if (sm.hist[s1] <= 64 && sm.hist[s2] <= 64) {
      pick_in_lists(sm, vals, n, sub, s1, s2, want2);
      *u1 = sm.pick[0];
      *u2 = want2 ? sm.pick[1] : sm.pick[0];
      return;
    }
    __syncthreads();   // every thread has read the second level's counts
  }
  *u1 = radix_select(vals, n, k, sm.scratch);
  *u2 = want2 ? radix_select(vals, n, k + 1, sm.scratch) : *u1;
}

// Inclusive prefix maximum over the wave of values >= -1.
__device__ __forceinline__ int wave_incl_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xA, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xC, 0xF, false));
  return v;
}

// The longest run of the n sorted values whose consecutive gaps stay below tau (the first of
// equal ones), as the rank of its first value and its length, without sorting: the values
// are counted in bins of 0.4 tau. Two neighbours a gap of tau or more apart lie at least
// two bins apart, so a run can only break across an empty bin, between the largest value
// of the last bin before it and the smallest of the first bin after it: only the bins
// beside an empty one need those two. False when the range takes more than 1024 bins
// (nothing written; sm.hist is then still all zero). All 256 threads; sm.hist zero on entry,
// used up on return.
//
// A sort of 2048 values in LDS takes 66 barriers; this takes eight. The 48 boxes of a
// 1080p frame with close blocks of 8 x 8 aggregate in 8.8 us instead of 30, the four of a
// 640 x 480 frame (up to 300 blocks each) in 7.1 instead of 9.6.
__device__ __forceinline__ bool longest_run(AggLds& sm, const float* vals, int n, float vmin, float vmax,
                                            float tau, int* start, int* len) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float scale = 2.5f / tau;
  if (!((vmax - vmin) * scale < 1023.0f)) return false;   // also tau = 0
  for (int i = tid; i < 1024; i += 256) {
    sm.lo[i] = 0x7FFFFFFFu;
    sm.hi[i] = 0u;
  }
  if (tid == 0) sm.run = 0;
  for (int i = tid; i < n; i += 256) atomicAdd(&sm.hist[value_bin(vals[i], vmin, scale)], 1);
  __syncthreads();
  for (int i = tid; i < n; i += 256) {
    const float v = vals[i];
    const int b = value_bin(v, vmin, scale);
    if (b == 1023 || sm.hist[b + 1] == 0) atomicMax(&sm.hi[b], __float_as_uint(v));
    if (b == 0 || sm.hist[b - 1] == 0) atomicMin(&sm.lo[b], __float_as_uint(v));
  }
  __syncthreads();
  // thread t owns bins 4t .. 4t + 3: the values before them and the last filled bin before them
  int c[4], sum = 0, last = -1;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c[k] = sm.hist[4 * tid + k];
    sum += c[k];
    if (c[k]) last = 4 * tid + k;
  }
  const int incl = wave_incl_scan(sum), mx = wave_incl_max(last);
  if (lane == 63) {
    sm.scratch[256 + wave] = incl;
    sm.scratch[260 + wave] = mx;
  }
  __syncthreads();
  int before = incl - sum;
  int prev = __builtin_amdgcn_update_dpp(-1, mx, 0x138, 0xF, 0xF, false);   // the lane before's
  for (int v = 0; v < wave; ++v) {
    before += sm.scratch[256 + v];
    prev = max(prev, sm.scratch[260 + v]);
  }
  // the first ranks of the runs that begin in the thread's bins
  int first[4], nb = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int b = 4 * tid + k;
    first[k] = -1;
    if (c[k]) {
      const bool brk = prev < 0 || (b - prev >= 2 && !(__uint_as_float(sm.lo[b]) - __uint_as_float(sm.hi[prev]) < tau));
      if (brk) {
        first[k] = before;
        ++nb;
      }
      prev = b;
    }
    before += c[k];
  }
  const int nincl = wave_incl_scan(nb);
  if (lane == 63) sm.scratch[264 + wave] = nincl;
  __syncthreads();
  int at = nincl - nb, runs = 0;
  for (int v = 0; v < kItemWaves; ++v) {
    if (v < wave) at += sm.scratch[264 + v];
    runs += sm.scratch[264 + v];
  }
  // their list, in order, over the counts
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (first[k] >= 0) sm.hist[at++] = first[k];
  __syncthreads();
  for (int j = tid; j < runs; j += 256) {
    const int l = (j + 1 < runs ? sm.hist[j + 1] : n) - sm.hist[j];
    atomicMax(&sm.run, ((unsigned long long)l << 32) | (0xFFFFFFFFu - (uint32_t)j));
  }
  __syncthreads();
  const unsigned long long r = sm.run;
  *len = (int)(r >> 32);
  *start = sm.hist[0xFFFFFFFFu - (uint32_t)r];
  return true;
}

__device__ __forceinline__ void aggregate_box(const MatchParamsDev& P, const MatchWs& ws, int kg,
                                              ocsr_box_result* out, bool timed_out, AggLds& sm) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const BoxPlan pl = ws.plan[kg];
  ocsr_box_result r = {};
  if (pl.status != -1 || timed_out) {
    if (tid == 0) {
      r.reason = timed_out ? OCSR_REASON_INTERNAL_TIMEOUT : pl.status;
      out[kg] = r;
    }
    return;
  }
  const int base = pl.frame * P.cap_blocks + pl.off;
  // a box of at most kAggMax blocks gathers its valid values into LDS; a larger one
  // compacts them in place at the front of its own block values in global memory (a
  // value moves to an index no larger than its own, and every chunk is loaded before
  // any of it is stored)
  const bool in_lds = pl.nblk <= kAggMax;
  // the rest runs with vals in LDS or in global memory, each instance with its pointer's
  // memory space known to the compiler (LDS reads rather than generic ones, whose
  // latency is that of a memory access)
  auto rest = [&](float* vals) {
    if (tid == 0) {
      sm.n_valid = 0;
      sm.n_eligible = 0;
      sm.vmin = 0x7FFFFFFFu;
      sm.vmax = 0;
    }
    for (int i = tid; i < 1024; i += 256) sm.hist[i] = 0;
    __syncthreads();
    uint32_t vlo = 0x7FFFFFFFu, vhi = 0;   // bit patterns of non-negative floats
    // gather the valid values: one LDS atomic per wave, positions from the ballot. Flags
    // and values of up to kGather blocks per thread are loaded before any is used.
    constexpr int kGather = 4;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int b0 = 0; b0 < pl.nblk; b0 += 256 * kGather) {
      uint32_t fl[kGather];
      float v[kGather];
  #pragma unroll
      for (int u = 0; u < kGather; ++u) {
        const int i = b0 + 256 * u + tid;
        const int at = base + (i < pl.nblk ? i : 0);
        fl[u] = ws.blk_flag[at];
        v[u] = ws.blk_val[at];
        fl[u] = i < pl.nblk ? fl[u] : 0u;
      }
      if (!in_lds) __syncthreads();   // the chunk is loaded before it is overwritten
  #pragma unroll
      for (int u = 0; u < kGather; ++u) {
        const uint64_t mv = __ballot((fl[u] & 2) != 0);
        const uint64_t me = __ballot((fl[u] & 1) != 0);
        int wbase = 0;
        if (lane == 0 && (mv | me)) {
          wbase = atomicAdd(&sm.n_valid, (int)__popcll(mv));
          atomicAdd(&sm.n_eligible, (int)__popcll(me));
        }
        wbase = __shfl(wbase, 0, 64);
        if (fl[u] & 2) {
          vals[wbase + __popcll(mv & below)] = v[u];
          vlo = min(vlo, __float_as_uint(v[u]));
          vhi = max(vhi, __float_as_uint(v[u]));
        }
      }
      if (!in_lds) __syncthreads();
    }
    vlo = wave_min_u32(vlo);
    vhi = (uint32_t)wave_max((int)vhi);
    if (lane == 0) {
      atomicMin(&sm.vmin, vlo);
      atomicMax(&sm.vmax, vhi);
    }
    if (!in_lds) __threadfence_block();   // compacted values visible to the workgroup
    __syncthreads();
    const int nv = sm.n_valid, ne = sm.n_eligible;
    r.n_blocks = pl.nblk;
    r.n_eligible = ne;
    r.n_valid = nv;
    if (ne == 0 || nv == 0) {
      if (tid == 0) {
        r.reason = ne == 0 ? OCSR_REASON_NO_ELIGIBLE_BLOCKS : OCSR_REASON_NO_VALID_BLOCKS;
        out[kg] = r;
      }
      return;
    }
    float d_box = 0.0f;
    bool ok = true;
    if (pl.level == 0 && pl.nblk == 1) {
      // Alg. 2: a FAR object matched as one block takes that block's result; CLOSE
      // objects always go through the robust aggregation
      d_box = vals[0];
      r.n_used = 1;
    } else if (P.agg_mode == OCSR_AGG_TRIMMED_MEDIAN) {
      // symmetric trim of floor(pct * n / 100) values at each end, then the median: the
      // one or two middle order statistics, found by selection
      const int t = P.trim_pct * nv / 100;
      const int m = nv - 2 * t;
      r.n_used = m > 0 ? m : 0;
      if (m <= 0 || m < P.n_min) {
        ok = false;
      } else {
        const int k1 = t + (m - 1) / 2;
        uint32_t u1, u2;
        select_middle(sm, vals, nv, k1, (m & 1) == 0, __uint_as_float(sm.vmin),
                      __uint_as_float(sm.vmax), &u1, &u2);
        d_box = (m & 1) ? __uint_as_float(u1) : (__uint_as_float(u1) + __uint_as_float(u2)) * 0.5f;
      }
    } else {
      const float vmin = __uint_as_float(sm.vmin), vmax = __uint_as_float(sm.vmax);
      int seg_start, seg_len;
      const bool binned = longest_run(sm, vals, nv, vmin, vmax, P.tau_d, &seg_start, &seg_len);
      if (!binned) {
        if (in_lds) {
          // bitonic sort of the valid values, padded with +inf to a power of two
          int n2 = 1;
          while (n2 < nv) n2 <<= 1;
          for (int i = nv + tid; i < n2; i += 256) sm.vals[i] = __builtin_inff();
          __syncthreads();
          for (int kk = 2; kk <= n2; kk <<= 1) {
            for (int j = kk >> 1; j > 0; j >>= 1) {
              for (int i = tid; i < n2; i += 256) {
                const int ixj = i ^ j;
                if (ixj > i) {
                  const float a = sm.vals[i], c = sm.vals[ixj];
                  const bool up = (i & kk) == 0;
                  if ((a > c) == up) { sm.vals[i] = c; sm.vals[ixj] = a; }
                }
              }
              __syncthreads();
            }
          }
        } else {
          // the values in global memory, ordered by a radix sort through the box's slots of
          // the sort buffer
          radix_sort_global(vals, ws.agg_tmp + base, nv, sm.hist, sm.scratch);
        }
        // longest run whose consecutive gaps stay below tau_d; the first run wins a tie
        if (tid < 64) {
          int best_start = 0, best_len = 1, start = 0;
          for (int b0 = 0; b0 < nv; b0 += 64) {
            const int q = b0 + tid;
            const bool brk = q > 0 && q < nv && !(vals[q] - vals[q - 1] < P.tau_d);
            uint64_t m = __ballot(brk);
            while (m) {
              const int pos = b0 + __ffsll((unsigned long long)m) - 1;
              m &= m - 1;
              const int len = pos - start;
              if (len > best_len) { best_len = len; best_start = start; }
              start = pos;
            }
          }
          const int len = nv - start;
          if (len > best_len) { best_len = len; best_start = start; }
          if (tid == 0) { sm.seg_start = best_start; sm.seg_len = best_len; }
        }
        __syncthreads();
        seg_start = sm.seg_start;
        seg_len = sm.seg_len;
      }
      r.n_used = seg_len;
      if (seg_len < P.n_min) {
        ok = false;
      } else if (!binned) {
        d_box = median_sorted(vals + seg_start, seg_len);
      } else {
        // the one or two middle order statistics of the run, among all values
        __syncthreads();   // every thread has read the run's list
        for (int i = tid; i < 1024; i += 256) sm.hist[i] = 0;
        __syncthreads();
        uint32_t u1, u2;
        select_middle(sm, vals, nv, seg_start + (seg_len - 1) / 2, (seg_len & 1) == 0, vmin, vmax, &u1, &u2);
        d_box = (seg_len & 1) ? __uint_as_float(u1) : (__uint_as_float(u1) + __uint_as_float(u2)) * 0.5f;
      }
    }
    if (tid == 0) {
      if (!ok) {
        r.reason = OCSR_REASON_TOO_FEW_CONSISTENT;
      } else {
        r.disparity = d_box;
        if (!(d_box > P.d_eps)) {
          r.reason = OCSR_REASON_NONPOSITIVE_DISPARITY;
        } else {
          r.depth = P.fb / d_box;   // Eq. 1, IEEE fp32 division
          r.valid = 1;
          r.reason = OCSR_REASON_OK;
        }
      }
      out[kg] = r;
    }
  };
  if (in_lds) rest(sm.vals);
  else rest(ws.blk_val + base);
}

// ---------------------------------------------------------------------------------
// Matchers of one level's blocks, for the level and pair kernels: the register-blocked
// kernel (ROWS block rows per wave, CPL candidates per lane, PASSES passes) and the generic
// kernel; those on the matrix cores are in dev_matrix.hpp.
// run_item: wave `wave`'s share of work item r (frame f, level `level`).
// frame_state: what a matcher reads per frame before an item's plan arrives (issued
// first, so that its loads and the plan's are in flight together).
struct NoFrameState {};
template <int ROWS, int NX, int CPL, int PASSES>
struct TiledMatcher {
  static constexpr size_t kLds = (Tiled<ROWS, NX, CPL, PASSES>::kLdsBytes + 15) & ~(size_t)15;
  static constexpr bool kShares = false;
  using State = NoFrameState;
  static __device__ __forceinline__ State frame_state(const MatchWs&, const FrameDev&, int) { return {}; }
  static __device__ __forceinline__ void run_item(const MatchParamsDev& P, const FrameDev& fr,
                                                  const MatchWs& ws, const DebugDev& dbg, int f,
                                                  int level, const ItemRec& r, int wave, int lane,
                                                  void* lds, const State& = State()) {
    run_item_rec(P, fr, f, level, r, wave, [&](const BlockCtx& c) {
      match_block_tiled<ROWS, NX, CPL, PASSES>(P, fr, ws, dbg, c, lane, lds);
    });
  }
};
// any block of up to 64 points (GRID blocks included), lanes over candidates
struct GenericMatcher {
  static constexpr size_t kLds = (kGenericLdsBytes + 15) & ~(size_t)15;
  static constexpr bool kShares = false;
  using State = NoFrameState;
  static __device__ __forceinline__ State frame_state(const MatchWs&, const FrameDev&, int) { return {}; }
  static __device__ __forceinline__ void run_item(const MatchParamsDev& P, const FrameDev& fr,
                                                  const MatchWs& ws, const DebugDev& dbg, int f,
                                                  int level, const ItemRec& r, int wave, int lane,
                                                  void* lds, const State& = State()) {
    run_item_rec(P, fr, f, level, r, wave, [&](const BlockCtx& c) {
      match_block_generic(P, fr, ws, dbg, c, lane, lds);
    });
  }
};
}  // namespace dev
}  // namespace ocsr
