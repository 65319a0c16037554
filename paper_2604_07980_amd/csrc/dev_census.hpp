// Census transform of one 64 x 32 tile of level pixels by one workgroup of 256
// threads (Sec. 4.3.1: census equation and Alg. 1).
//
// The tile plus its halo is staged in LDS as bytes. Each lane owns four horizontally
// adjacent pixels of two rows, a pixel per byte of a word, and compares four at once:
// v_lerp_u8 of a neighbour word and the complemented centre word, (n + 255 - c) >> 1 in
// every byte, has bit 7 set exactly where the neighbour is brighter. A shift and a bit-field
// insert file the four bits in a running word, eight comparisons to a byte of the code, and
// byte permutes put the eight bytes of each pixel's code together: three VALU instructions
// for four comparisons, counted over the kernel 1.10 per comparison, against 1.28 with
// 16-bit subtracts of two pixels. Both the VALU (10.5 us of it for a 1080p pair at two
// levels) and the stores (8.5 us for its 42 MB at the rate of a fill) bound it: the pair takes
// 15.8 us (17.1 with the subtracts), the 138 MB of 16 listed 1200p frames 48.8 us (54.5).
//
// Bit order: Alg. 1 starts from the sentinel and, for i = -SX..SX (x, outer) and
// j = -SY..SY (y, inner), shifts left and appends [I(x+i, y+j) > I(x, y)]; the first
// comparison therefore ends at bit n-1 (n = (2SX+1)(2SY+1)) and the sentinel at bit n.
// Pixels whose window leaves the level image store 0.
#pragma once

#include "dev_common.hpp"

namespace ocsr {
namespace dev {

// alignment of the LDS that a tile is made in
constexpr size_t kCensusLdsAlign = 16;

constexpr int kCensusRowsPerLane = 2;   // 4 waves x 4 lane groups x 2 rows = kCensusTileY

template <int SX, int SY>
struct CensusTile {
  static constexpr int LW = (kCensusTileX + 2 * SX + 3) / 4;      // words of a staged row
  static constexpr int LP = 24;                                   // LDS words per row: the four lane
                                                                  // groups of a wave, two rows
                                                                  // apart, read different banks
  static constexpr int LR = kCensusTileY + 2 * SY;                // staged rows
  static constexpr int N = (2 * SX + 1) * (2 * SY + 1);           // comparisons
  // the staged tile, then 512 words per wave in which a row of codes changes lanes
  static constexpr int kOutAt = LP * LR;
  static constexpr size_t kLdsBytes = sizeof(uint32_t) * (kOutAt + 4 * 512);
  static_assert(N + 1 <= 64, "window wider than a 64-bit code");
  static_assert(kOutAt % 4 == 0, "codes change lanes in 16-byte accesses (kCensusLdsAlign)");
  static_assert(SX <= 4 && LW <= LP, "a lane's window row is at most three words");
};

// One census tile: the uint8 source img (pitch bytes, W x H) at level scale s (level
// image Ws x Hs = W/s x H/s), the level position (X0, Y0) of the tile, and the
// descriptor image out (out_pitch words).
struct CensusJob {
  const uint8_t* img;
  int W, H, pitch, s, Ws, Hs;
  uint64_t* out;
  int out_pitch, X0, Y0;
};

// Word (r, c) of the staged tile is level samples 4c .. 4c + 3 of row r, counted from the
// halo's corner. A position outside the level image reads some valid byte of the image
// instead: only pixels whose window leaves the image see such values, and their words are
// stored as 0 regardless.
__device__ __forceinline__ int clamp_to(int v, int n) { return v < 0 ? 0 : (v < n ? v : n - 1); }

// y moved down by one bit with bit 7 of every byte of x on top: two instructions. m: 0x80808080
// in a vector register (v_bitop3_b32 and right shifts issue up to 1.6 times as fast as
// other three-operand instructions, but only without scalar operands). As asm: free to
// reassociate the builtin, the compiler takes 84 registers instead of 50 and loses half the
// waves.
__device__ __forceinline__ uint32_t push_bits(uint32_t y, uint32_t x, uint32_t m) {
  uint32_t r;                                   // m ? x : y >> 1
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0xca" : "=v"(r) : "v"(m), "v"(x), "v"(y >> 1));
  return r;
}

// Whether tile j's samples are read as words (level scales 1 and 2): every staged sample, and
// four more to the right, lies inside the level image. Uniform over the workgroup.
template <int SX, int SY>
__device__ __forceinline__ bool census_words(const CensusJob& j) {
  using T = CensusTile<SX, SY>;
  return uniform(j.s <= 2 && j.X0 >= SX && j.X0 - SX + 4 * T::LW + 4 <= j.Ws && j.Y0 >= SY &&
                 j.Y0 - SY + T::LR <= j.Hs) != 0;
}

// Stages tile j in P. A tile of words takes eight unaligned bytes per staged word (at scale 1
// the first four are the word, at scale 2 the even ones); the others (on the image's border,
// or at other scales) a clamped byte per sample. All loads are issued before the first is
// waited for. Called by all 256 threads of the workgroup.
template <int SX, int SY>
__device__ __forceinline__ void census_stage(const CensusJob& j, uint32_t* P) {
  using T = CensusTile<SX, SY>;
  constexpr int NT = T::LW * T::LR, NW = (NT + 255) / 256;
  const int s = uniform(j.s);
  const int64_t pitch = (int64_t)s * uniform(j.pitch);   // of a level row
  const uint8_t* img = uniform(j.img);
  const int X0 = uniform(j.X0) - SX, Y0 = uniform(j.Y0) - SY;
  // thread t stages the words t, t + 256, .. (threads past the tile its last word again)
  if (census_words<SX, SY>(j)) {
    const uint8_t* corner = img + Y0 * pitch + s * X0;
    const uint32_t sel = s == 1 ? 0x03020100u : 0x06040200u;
    uint64_t w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int t = min((int)threadIdx.x + 256 * i, NT - 1);
      const int r = t / T::LW, c = t - r * T::LW;
      __builtin_memcpy(&w[i], corner + r * pitch + 4 * s * c, 8);
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int t = min((int)threadIdx.x + 256 * i, NT - 1);
      const int r = t / T::LW, c = t - r * T::LW;
      P[r * T::LP + c] = __builtin_amdgcn_perm((uint32_t)(w[i] >> 32), (uint32_t)w[i], sel);
    }
  } else {
    const int Ws = uniform(j.Ws), Hs = uniform(j.Hs);
    uint32_t b[NW][4];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int t = min((int)threadIdx.x + 256 * i, NT - 1);
      const int r = t / T::LW, c = t - r * T::LW;
      const uint8_t* row = img + clamp_to(Y0 + r, Hs) * pitch;
#pragma unroll
      for (int k = 0; k < 4; ++k) b[i][k] = row[s * clamp_to(X0 + 4 * c + k, Ws)];
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int t = min((int)threadIdx.x + 256 * i, NT - 1);
      const int r = t / T::LW, c = t - r * T::LW;
      P[r * T::LP + c] = b[i][0] | (b[i][1] << 8) | (b[i][2] << 16) | (b[i][3] << 24);
    }
  }
}

// The census words of tile j from P (staged by census_stage), after a barrier. Called
// by all 256 threads of the workgroup.
template <int SX, int SY>
__device__ __forceinline__ void census_compute(const CensusJob& j, int sentinel, uint32_t* P) {
  using T = CensusTile<SX, SY>;
  constexpr int R = kCensusRowsPerLane, LP = T::LP, N = T::N;
  constexpr int WR = R + 2 * SY;                // staged rows a lane reads
  uint64_t* out = uniform(j.out);
  const int out_pitch = uniform(j.out_pitch);
  const int X0 = uniform(j.X0), Y0 = uniform(j.Y0);
  const int Ws = uniform(j.Ws), Hs = uniform(j.Hs);
  const int tid = threadIdx.x;
  const int col = tid & 15, r0 = R * (tid >> 4);
  // the lane's window: words col .. col + 2 of WR rows (bytes 0 .. 3 + 2 SX)
  uint32_t d[WR][3];
  const uint32_t* Pl = P + r0 * LP + col;
#pragma unroll
  for (int r = 0; r < WR; ++r)
#pragma unroll
    for (int k = 0; k < 3; ++k) d[r][k] = 4 * k < 4 + 2 * SX ? Pl[r * LP + k] : 0u;
  const uint32_t m = in_vgpr(0x80808080u);
  const bool inside = X0 >= SX && X0 + kCensusTileX <= Ws - SX && Y0 >= SY && Y0 + kCensusTileY <= Hs - SY;
  // four pixels of staged row r, i columns right of the window's left edge
  auto window = [&](int r, int i) {
    return (i & 3) == 0 ? d[r][i >> 2] : __builtin_amdgcn_alignbyte(d[r][min((i >> 2) + 1, 2)], d[r][i >> 2], i & 3);
  };
  uint32_t nc[R];                               // the complemented centres
#pragma unroll
  for (int k = 0; k < R; ++k) nc[k] = ~window(SY + k, SX);
  // code byte q of the four pixels of each row; y collects a byte's bits from bit 7 down:
  // each new one goes to bit 7 after the others moved down (what crosses into the next
  // pixel's bit 7 is overwritten by the same step). Window column by window column for both
  // rows, which share the shifted words (row by row they stay in 40 more registers).
  uint32_t code[R][8], y[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    y[k] = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) code[k][q] = 0;
  }
#pragma unroll
  for (int i = 2 * SX; i >= 0; --i) {
    uint32_t v[WR];
#pragma unroll
    for (int r = 0; r < WR; ++r) v[r] = window(r, i);
#pragma unroll
    for (int jj = 2 * SY; jj >= 0; --jj) {
      const int pos = N - 1 - (i * (2 * SY + 1) + jj);   // Alg. 1 order, MSB first
#pragma unroll
      for (int k = 0; k < R; ++k) {
        if (i == SX && jj == SY) {              // the centre against itself: its bit is 0
          y[k] = (pos & 7) == 0 ? 0u : (y[k] >> 1) & 0x7F7F7F7Fu;
        } else {
          const uint32_t x = __builtin_amdgcn_lerp(v[jj + k], nc[k], 0u);
          y[k] = (pos & 7) == 0 ? x : push_bits(y[k], x, m);
        }
        if ((pos & 7) == 7) code[k][pos >> 3] = y[k];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    // the sentinel above the last comparison, and the top byte's bits moved to its low end
    {
      constexpr int top = N & 7;                // the sentinel's bit
      const uint32_t sb = sentinel ? 0x80808080u : 0u;
      uint32_t t = top == 0 ? sb : sb | ((y[k] >> 1) & 0x7F7F7F7Fu);
      if (top < 7) t = (t >> (7 - top)) & (0x01010101u * ((1u << (top + 1)) - 1u));
      code[k][N >> 3] = t;
    }
    // 4 x 4 byte transposes: word h of pixel p's code
    uint32_t w[4][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t* c = code[k] + 4 * h;
      const uint32_t a0 = __builtin_amdgcn_perm(c[1], c[0], 0x05010400u), a1 = __builtin_amdgcn_perm(c[1], c[0], 0x07030602u);
      const uint32_t b0 = __builtin_amdgcn_perm(c[3], c[2], 0x05010400u), b1 = __builtin_amdgcn_perm(c[3], c[2], 0x07030602u);
      w[0][h] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
      w[1][h] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
      w[2][h] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
      w[3][h] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
    }
    if (inside) {
      // through LDS, so that a store covers two whole rows of 512 bytes, 16 bytes a lane
      // (straight from the lanes it would cover every other 16 bytes of four rows, which
      // writes at 4.0 TB/s where whole rows reach 5.0)
      const int lane = tid & 63, wave = tid >> 6;
      uint32_t* o = P + T::kOutAt + wave * 512;
      wave_sync();                              // the previous row is read
      *(uint4*)(o + 8 * lane) = uint4{w[0][0], w[0][1], w[1][0], w[1][1]};
      *(uint4*)(o + 8 * lane + 4) = uint4{w[2][0], w[2][1], w[3][0], w[3][1]};
      wave_sync();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // lane l holds 16 bytes of the wave's row group 2 h + l / 32
        const uint4 v = *(const uint4*)(o + 256 * h + 4 * lane);
        const int Y = Y0 + R * (4 * wave + 2 * h + (lane >> 5)) + k;
        __builtin_memcpy(out + (size_t)Y * out_pitch + X0 + 2 * (lane & 31), &v, 16);
      }
    } else {
      const int Y = Y0 + r0 + k, X = X0 + 4 * col;
      if (Y < Hs) {
        uint64_t* o = out + (size_t)Y * out_pitch + X;
        const bool row_def = Y >= SY && Y < Hs - SY;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          if (X + p < Ws) {
            const bool def = row_def && X + p >= SX && X + p < Ws - SX;
            o[p] = def ? ((uint64_t)w[p][1] << 32) | w[p][0] : 0ull;
          }
        }
      }
    }
  }
}

// One tile, staged through registers.
template <int SX, int SY>
__device__ __forceinline__ void census_tile(const uint8_t* __restrict__ img, int W, int H,
                                            int pitch, int s, uint64_t* __restrict__ out,
                                            int out_pitch, int X0, int Y0, int sentinel,
                                            uint32_t* P) {
  const CensusJob j{img, W, H, pitch, s, W / s, H / s, out, out_pitch, X0, Y0};
  census_stage<SX, SY>(j, P);
  __syncthreads();
  census_compute<SX, SY>(j, sentinel, P);
}

// Any window: one pixel per thread per row, straight from global memory (no LDS).
__device__ __forceinline__ void census_tile_generic(const uint8_t* __restrict__ img, int W, int H,
                                                    int pitch, int s, uint64_t* __restrict__ out,
                                                    int out_pitch, int X0, int Y0, int sx, int sy,
                                                    int sentinel) {
  const int Ws = W / s, Hs = H / s;
  const int X = X0 + (threadIdx.x & 63);
  for (int Y = Y0 + (int)(threadIdx.x >> 6); Y < Y0 + kCensusTileY; Y += 4) {
    if (X >= Ws || Y >= Hs) continue;
    uint64_t code = 0;
    if (X >= sx && X < Ws - sx && Y >= sy && Y < Hs - sy) {
      const uint8_t c = img[(size_t)(s * Y) * pitch + (size_t)(s * X)];
      code = sentinel ? 1ull : 0ull;
      for (int i = -sx; i <= sx; ++i)
        for (int j = -sy; j <= sy; ++j) {
          const uint8_t n = img[(size_t)(s * (Y + j)) * pitch + (size_t)(s * (X + i))];
          code = (code << 1) | (n > c ? 1ull : 0ull);
        }
    }
    out[(size_t)Y * out_pitch + X] = code;
  }
}

// Whether a box's search reads some pixel of the census tile [X0, X0 + 64) x
// [Y0, Y0 + 32) of one view at one level. A ranged box belongs to the level of its
// far/close type (Sec. 4.3.4); its blocks lie in the level rectangle [x0, x1) x [y0, y1)
// of its eligible pixels (the same clipping as the plan). With candidates dlo..dhi, the
// forward search reads the right view on [x0 - dhi, x1 - dlo); the template and the
// backward search read the left view on [x0 - (dhi - dlo), x1 + (dhi - dlo)); all on
// rows [y0, y1). The loop and the result are uniform over the wave.
__device__ __forceinline__ bool census_tile_needed(const MatchParamsDev& MP, const FrameDev& fr,
                                                   const ocsr_box* __restrict__ boxes, int level,
                                                   int view, int X0, int Y0) {
  const int lane = threadIdx.x & 63;
  const LevelDev& lv = fr.lv[level];
  const int s = lv.scale;
  const int dlo = MP.path[level].dlo, dhi = dlo + MP.path[level].nd - 1;
  const int ext_lo = view ? dhi : dhi - dlo;   // the read range starts this far left of x0
  const int ext_hi = view ? -dlo : dhi - dlo;  // and ends this far right of x1
  // rows: the right view is read at y + dy, the left view (backward) at y + dy_f - dy
  const int eylo = MP.path[level].dylo, eyhi = eylo + MP.path[level].ndy - 1;
  const int ey_lo = view ? -eylo : eyhi - eylo;  // rows start this far above y0
  const int ey_hi = view ? eyhi : eyhi - eylo;   // and end this far below y1
  for (int base = 0; base < fr.n_boxes; base += 64) {
    const int i = base + lane;
    bool hit = false;
    if (i < fr.n_boxes) {
      const ocsr_box b = boxes[fr.box_off + i];
      const int cx0 = max(b.x0, 0), cy0 = max(b.y0, 0);
      const int cx1 = min(b.x1, fr.W), cy1 = min(b.y1, fr.H);
      if ((b.flags & OCSR_BOX_RANGE) && cx0 < cx1 && cy0 < cy1 &&
          (max(cx1 - cx0, cy1 - cy0) < MP.tau_s ? 0 : 1) == level) {
        const int x0 = max(cdiv_nonneg(cx0, s), lv.sx), x1 = min(cdiv_nonneg(cx1, s), lv.W - lv.sx);
        const int y0 = max(cdiv_nonneg(cy0, s), lv.sy), y1 = min(cdiv_nonneg(cy1, s), lv.H - lv.sy);
        hit = x0 < x1 && y0 < y1 && y0 - ey_lo < Y0 + kCensusTileY && Y0 < y1 + ey_hi &&
              x0 - ext_lo < X0 + kCensusTileX && X0 < x1 + ext_hi;
      }
    }
    if (__ballot(hit)) return true;
  }
  return false;
}

// Census tile c of a whole-frame call: the tiles of frame f start at
// FR.f[f].tile_begin and run over view L then R at level 1, then L and R at level 0.
// Level 1 comes first: its tiles are few and mostly read by the close boxes, so they are
// dispatched ahead of the many, mostly skipped, tiles of level 0.
struct FrameTile {
  int f, level, view;
  CensusJob job;
};
// Frame-local tile t of frame f (the frame's tiles number fewer than 2^30; the row of a
// tile comes from the frame's reciprocal of its tiles per row, without a division).
__device__ __forceinline__ FrameTile frame_tile_local(const FrameDev& fr, int f, int t) {
  int level = 1, tiles = fr.tiles1, tiles_x = fr.tiles1_x;
  uint64_t recip = fr.tx_recip[1];
  if (t >= 2 * fr.tiles1) {
    t -= 2 * fr.tiles1;
    level = 0;
    tiles = fr.tiles0;
    tiles_x = fr.tiles0_x;
    recip = fr.tx_recip[0];
  }
  const int view = t >= tiles ? 1 : 0;
  t -= view ? tiles : 0;
  const int ty = (int)(((uint64_t)(uint32_t)t * recip) >> 40);
  const int tx = t - ty * tiles_x;
  const LevelDev& lv = fr.lv[level];
  FrameTile ft;
  ft.f = f;
  ft.level = level;
  ft.view = view;
  ft.job = CensusJob{view ? fr.imgR : fr.imgL, fr.W, fr.H, fr.pitch, lv.scale, lv.W, lv.H,
                     (uint64_t*)(view ? lv.R : lv.L), lv.pitch, tx * kCensusTileX, ty * kCensusTileY};
  return ft;
}
__device__ __forceinline__ FrameTile frame_tile(const FramesDev& FR, int c) {
  int f = 0;
  for (int k = 1; k < FR.n; ++k)
    if (c >= FR.f[k].tile_begin) f = k;
  return frame_tile_local(FR.f[f], f, c - FR.f[f].tile_begin);
}

// Makes tile j: window (SX, SY) > (-1, -1) through LDS, (-1, -1) the generic code with
// (sx, sy). All 256 threads of the workgroup.
template <int SX, int SY>
__device__ __forceinline__ void make_census_tile(const CensusJob& j, int sx, int sy, int sentinel,
                                                 uint32_t* P) {
  if constexpr (SX >= 0) {
    census_stage<SX, SY>(j, P);
    __syncthreads();
    census_compute<SX, SY>(j, sentinel, P);
  } else {
    census_tile_generic(j.img, j.W, j.H, j.pitch, j.s, j.out, j.out_pitch, j.X0, j.Y0, sx, sy, sentinel);
  }
}

// Makes census tile c of a whole-frame call. With `check` set and MP.full_census clear,
// a tile no box's search reads is skipped (every wave of the workgroup takes the same
// decision). Window (SX, SY) > (-1, -1) takes the LDS code; (-1, -1) the generic code
// with (sx, sy).
template <int SX, int SY>
__device__ __forceinline__ void frame_census_tile(const MatchParamsDev& MP, const FramesDev& FR,
                                                  const ocsr_box* __restrict__ boxes, int c,
                                                  int sx, int sy, int sentinel, uint32_t* P,
                                                  bool check = true, int* verdict = nullptr) {
  const FrameTile ft = frame_tile(FR, c);
  const CensusJob& j = ft.job;
  if (check && !MP.full_census) {
    const FrameDev& fr = FR.f[ft.f];
    bool needed;
    if (verdict) {
      // wave 0 tests the tile and shares the verdict through LDS (verdict must not alias P)
      if (threadIdx.x < 64) {
        const bool v = census_tile_needed(MP, fr, boxes, ft.level, ft.view, j.X0, j.Y0);
        if (threadIdx.x == 0) *verdict = v ? 1 : 0;
      }
      __syncthreads();
      needed = *verdict != 0;
    } else {
      needed = census_tile_needed(MP, fr, boxes, ft.level, ft.view, j.X0, j.Y0);
    }
    if (!needed) return;
  }
  make_census_tile<SX, SY>(j, sx, sy, sentinel, P);
}

// Sets, in bits, the tile bits of the frame's boxes (thread t0 of nt threads; atomic ORs,
// so threads may share a map). With fewer boxes than threads, tpb threads share a box and
// take every tpb-th of its tile rows: thread t0 takes boxes t0 / tpb, t0 / tpb + nt / tpb,
// ... and rows sub, sub + tpb, ... of each.
__device__ __forceinline__ void mark_frame_tiles(const MatchParamsDev& MP, const FrameDev& fr,
                                                 const ocsr_box* __restrict__ boxes,
                                                 uint32_t* bits, int t0, int nt) {
  const int tpb = max(1, min(8, nt / max(fr.n_boxes, 1)));
  const int sub = t0 % tpb, groups = nt / tpb;
  if (t0 >= groups * tpb) return;
  for (int i = t0 / tpb; i < fr.n_boxes; i += groups) {
    const ocsr_box b = boxes[fr.box_off + i];
    const int cx0 = max(b.x0, 0), cy0 = max(b.y0, 0);
    const int cx1 = min(b.x1, fr.W), cy1 = min(b.y1, fr.H);
    if (!(b.flags & OCSR_BOX_RANGE) || !(cx0 < cx1 && cy0 < cy1)) continue;
    const int level = max(cx1 - cx0, cy1 - cy0) < MP.tau_s ? 0 : 1;
    const LevelDev& lv = fr.lv[level];
    const int s = lv.scale;
    const int x0 = max(cdiv_nonneg(cx0, s), lv.sx), x1 = min(cdiv_nonneg(cx1, s), lv.W - lv.sx);
    const int y0 = max(cdiv_nonneg(cy0, s), lv.sy), y1 = min(cdiv_nonneg(cy1, s), lv.H - lv.sy);
    if (!(x0 < x1 && y0 < y1)) continue;
    const int dlo = MP.path[level].dlo, dhi = dlo + MP.path[level].nd - 1;
    const int eylo = MP.path[level].dylo, eyhi = eylo + MP.path[level].ndy - 1;
    const int tiles_x = level ? fr.tiles1_x : fr.tiles0_x;
    const int tiles = level ? fr.tiles1 : fr.tiles0;
    const int tiles_y = tiles / tiles_x;
    const int lbase = level ? 0 : 2 * fr.tiles1;
    for (int view = 0; view < 2; ++view) {
      const int a = max(x0 - (view ? dhi : dhi - dlo), 0);
      const int e = min(x1 + (view ? -dlo : dhi - dlo), tiles_x * kCensusTileX);
      if (a >= e) continue;
      const int ta = a / kCensusTileX, tb = (e - 1) / kCensusTileX;
      const int ya = max(y0 + (view ? eylo : eylo - eyhi), 0);
      const int yb = min(y1 + (view ? eyhi : eyhi - eylo), tiles_y * kCensusTileY);
      if (ya >= yb) continue;
      for (int ty = ya / kCensusTileY + sub; ty <= (yb - 1) / kCensusTileY; ty += tpb) {
        const int first = lbase + view * tiles + ty * tiles_x + ta;
        const int last = first + (tb - ta);
        for (int wd = first >> 5; wd <= (last >> 5); ++wd) {
          const int lo = max(first - 32 * wd, 0), hi = min(last - 32 * wd, 31);
          const uint32_t upto = hi == 31 ? 0xFFFFFFFFu : ((1u << (hi + 1)) - 1u);
          atomicOr(&bits[wd], upto & ~((1u << lo) - 1u));
        }
      }
    }
  }
}

// Word i of an empty tile map of n_tiles tiles, or of a full one with MP.full_census.
__device__ __forceinline__ uint32_t tile_map_init(const MatchParamsDev& MP, int n_tiles, int i) {
  const int rem = n_tiles - 32 * i;
  return !MP.full_census ? 0u : rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
}

// Writes the tiles set in the OR of n_maps maps (map m at bits + m * stride words) to
// fr.tile_list in increasing tile number and their number to the frame's FC_TILES
// counter. All 256 threads of the workgroup, after the maps are complete; sc: 8 ints.
__device__ __forceinline__ void compact_frame_tiles(const FrameDev& fr, int f, const MatchWs& ws,
                                                    const uint32_t* bits, int n_maps, int stride,
                                                    int* sc) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tiles = 2 * (fr.tiles0 + fr.tiles1);
  const int n_words = (n_tiles + 31) >> 5;
  auto word = [&](int i) {
    uint32_t m = 0;
    for (int k = 0; k < n_maps; ++k) m |= bits[k * stride + i];
    return m;
  };
  // thread t owns words [t wpt, (t + 1) wpt); ranks run in word order
  const int wpt = (n_words + 255) >> 8;
  const int w0 = tid * wpt;
  int cnt = 0;
  for (int k = 0; k < wpt; ++k)
    if (w0 + k < n_words) cnt += __popc(word(w0 + k));
  const int incl = wave_incl_scan(cnt);
  if (lane == 63) sc[wave] = incl;
  __syncthreads();
  int r = incl - cnt;
  for (int v = 0; v < wave; ++v) r += sc[v];
  for (int k = 0; k < wpt; ++k) {
    uint32_t m = w0 + k < n_words ? word(w0 + k) : 0u;
    while (m) {
      const int bit = __ffs(m) - 1;
      m &= m - 1;
      fr.tile_list[r++] = 32 * (w0 + k) + bit;
    }
  }
  if (tid == 255) ws.fcount[f * FC_N + FC_TILES] = r;
}

// The plan step's list of the census tiles of frame f: every tile some ranged box's
// search reads (the ranges of census_tile_needed), or every tile with MP.full_census,
// in increasing frame-local tile number (the order frame_census_tile decodes: level 1,
// view L then R, then level 0), written to fr.tile_list; their number to the frame's
// FC_TILES counter. One workgroup of 256 threads; bits: kFrameTileWords words of LDS,
// sc: 8 ints. The frame's tiles must number at most 32 kFrameTileWords.
__device__ __forceinline__ void list_frame_tiles(const MatchParamsDev& MP, const FrameDev& fr, int f,
                                                 const ocsr_box* __restrict__ boxes,
                                                 const MatchWs& ws, uint32_t* bits, int* sc) {
  const int tid = threadIdx.x;
  const int n_tiles = 2 * (fr.tiles0 + fr.tiles1);
  const int n_words = (n_tiles + 31) >> 5;
  for (int i = tid; i < n_words; i += 256) bits[i] = tile_map_init(MP, n_tiles, i);
  __syncthreads();
  if (!MP.full_census) {
    mark_frame_tiles(MP, fr, boxes, bits, tid, 256);
    __syncthreads();
  }
  compact_frame_tiles(fr, f, ws, bits, 1, 0, sc);
}

}  // namespace dev
}  // namespace ocsr
