// Dense counterpart of the object-centric path: every pixel, every disparity. Not part
// of the paper's method; it is the dense matcher the object-centric path is measured
// against (same census descriptors, same Hamming cost).
//
//   C(x, y, d)  = sum over the (2R+1)^2 window around (x, y), clipped to the image, of
//                 popcount(CL(x', y') ^ CR(x' - d, y'))   (CR is 0 outside the image)
//   d_L(x, y)   = smallest d in [dmin, dmax] minimising C(x, y, d)
//   d_R(xr, y)  = smallest d minimising C(xr + d, y, d) over d with xr + d inside
//   disp(x, y)  = d_L if x - d_L >= 0 and |d_L - d_R(x - d_L, y)| <= lr_tol, else -1
//
// A term is a dot product: with bit b of a word written as the sign (-1)^b of a one-digit
// number, popcount(p ^ q) = (64 - p . q) / 2. The matrix cores take such words as 64 FP4
// numbers of value +-1, so one 32 x 32 x 64 product gives the terms of 32 x 32 pairs of
// columns at 128 operations each (6 PFLOP/s measured, five times the rate of the vector
// ALU's two XORs and two popcounts). Sums of +-1 are exact in the fp32 accumulators.
//
// One wave per strip of `cols` output columns of the left view and band of kBand output rows.
// The strip's columns (32 with the window's halo) are the product's columns, one per lane; the
// right image's columns are its rows: a lane half holds 16 T consecutive ones in its
// accumulators, so a chunk of the search is 2 (16 T - 2R) candidate columns. The accumulators
// hold the vertical window sums: each step adds the products of the entering row and
// subtracts those of the leaving one (the leaving row's signs flipped). The horizontal window
// runs along a diagonal: the neighbour column in the next lane pairs with the next
// accumulator, so 2R wave-wide DPP adds of packed pairs of 16-bit sums finish a window. A
// candidate's key is cost << 4 | rank in 16 bits (cost << 3 with R = 3), two to a word: the
// digits are of magnitude 2 and 4, so that the sums come out of the products shifted. Packed
// minima run over 16 candidates (8 with R = 3) before they widen to cost << 16 | (d - dmin).
// Candidates outside the search range carry bit 15.
//
// The same costs give the right winners: those of a right column lie in one accumulator of
// every lane, so the keys (with the lane's rank in place of the accumulator's) turn through
// LDS, a lane takes a right column's 32, and the least goes to the column's word in memory by
// an atomic minimum, where the strips that see the column meet.
//
// Bound: vector ALU (packing, 2R adds, left and right key and minimum: 2R + 5 per two
// candidates; it issues in 86% of the cycles, the matrix cores are busy in 13%). Measured on a
// 1920 x 1080 pair with 192 candidates, R = 2: 169 us with the check, against 225 with a pass
// of its own for the right winners and 813 for the vector ALU alone (two XORs, two popcounts
// and about six more operations a term); on a 960 x 128 region of nine offsets 63 us against
// 78 and 262. Bands of 10 rows measure 1.5% less on the first and 2% more on the second, of 6
// rows 2% and 10% more; two waves per SIMD instead of three measure 10% more; the
// atomics cost 2%.
#include <algorithm>

#include "dev_fp4.hpp"

namespace ocsr {
namespace {

constexpr int kBand = 8;     // output rows per wave

struct DenseArgs {
  const uint64_t* CL;
  const uint64_t* CR;
  int32_t W, H, pitch;        // descriptor image size and row pitch (words)
  int32_t dlo, nd;            // disparities dlo .. dlo + nd - 1
  int32_t d_out;              // dmin, which the winners' indices are added to (dlo is at most
                              // W + 512: from W on every candidate's word lies outside)
  int16_t* left;              // [H][W] left winners' disparity (-1: no candidate)
  uint32_t* right;            // [H][W] right winners: d - dlo in the low half, above it the cost
                              // or (dense_few_kernel) nothing; kNoKey: no candidate
  // several pairs in one launch (grid z): pair z reads CL + z * cl_zstride (words; the
  // right image is shared) and writes left and right + z * out_zstride
  int64_t cl_zstride, out_zstride;
  int32_t cols, chunks;       // output columns per wave, chunks of the search
  int32_t strips, bands;      // of a pair
};

constexpr uint32_t kNoKey = 0xFFFFFFFFu;

using namespace dev;

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t shr1(uint32_t v) {   // lane i gets lane i - 1
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);
}

// The words of one image row that a chunk reads: the lane's fixed column and its T moving
// columns, 32 bits each (lanes 32..63 the high halves).
template <int T>
struct DenseRow {
  uint32_t f, m[T];
};

// How the right winners' keys change lanes: row h Z2 + z of LDS holds accumulator z of lane
// half h (packed with z + Z2) for the strip's 32 columns; 36 words a row, so that 16-byte
// reads of 16 rows hit all banks.
template <int T>
struct DenseTurn {
  static constexpr int Z2 = 8 * T, ROWS = 2 * Z2, STRIDE = 36;
  static constexpr int WORDS = ROWS * STRIDE;
};

template <int R>
constexpr int rank_bits() { return R == 3 ? 3 : 4; }
// every key of a valid candidate is below this, every other one above
template <int R>
constexpr uint32_t none_from() { return (0x8000u << (16 - rank_bits<R>())) - 0x10000u; }

template <int R, int T>
__device__ __forceinline__ void dense_chunk(const DenseArgs& a, int xs, int y0, int chunk, int lane,
                                            uint32_t* __restrict__ keys, uint32_t* __restrict__ turn) {
  constexpr int NW = 2 * R + 1;                 // window rows and columns
  constexpr int NR = kBand + 2 * R;             // rows walked
  constexpr int HS = 16 * T - 2 * R;            // candidate columns of a lane half
  constexpr int Z2 = 8 * T;                     // accumulators z and z + Z2 share a packed word
  constexpr int IB = rank_bits<R>();            // rank bits of a 16-bit key
  // the digits' magnitudes: a term adds 2^(IB - 1) times (64 - p . q), so that the sums are
  // keys already but for the rank
  constexpr uint32_t kFixed = R == 3 ? kTwo : kFour, kMoving = kTwo;
  constexpr float kTerms = 64.0f * (1 << (IB - 1)) * NW;
  constexpr int RUN = 1 << IB, NRUN = (Z2 + RUN - 1) / RUN;
  const int n = lane & 31, h = lane >> 5;
  const int W = a.W;
  const int x = xs + n - R;                     // the lane's fixed column
  const int c = xs + n - 2 * R;                 // centre of the window that ends in lane n
  // accumulator z of lane half h is moving column q0 + h HS + z (a window's last column)
  const int q0 = xs - (a.dlo + a.nd - 1) + 2 * HS * chunk - R;
  // loads: lane l gives row l & 31 of a product's first operand, whose accumulators are
  // those of lane half (m >> 2) & 1 at 4 (m >> 3) + (m & 3)
  const int qm = q0 + ((n >> 2) & 1) * HS + 4 * (n >> 3) + (n & 3);
  const uint32_t foff = 8u * (uint32_t)x + 4u * (uint32_t)h;
  const uint32_t sign = in_vgpr(kSign), mag = in_vgpr(kMoving);
  uint32_t moff[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int q = qm + 16 * t;
    moff[t] = q >= 0 && q < W ? 8u * (uint32_t)q + 4u * (uint32_t)h : ~7u;   // ~7: past any row
  }
  // terms count where the left column is inside; a word of the right image outside it is 0
  const bool f_in = x >= 0 && x < W;
  const uint32_t fsign = f_in ? kSign : 0u, fmag = f_in ? kFixed : 0u;
  // rank of each candidate within its run (smaller d first), bit 15 where d is outside
  // the range or the lane's window is not one of the strip's output columns
  // (accumulators z0 .. z1 hold valid candidates; bits of the others)
  uint32_t pen[Z2];
  {
    const int qc0 = q0 + h * HS - R;            // accumulator 0's centre
    const int k0 = c - a.dlo - (a.nd - 1) - qc0;   // first candidate
    const bool c_out = n >= 2 * R && n < 2 * R + a.cols && c < W;
    const int z0 = max(k0, 2 * R);
    const int z1 = c_out ? k0 + a.nd - 1 : -1;
    auto bits_from = [](int z) {                // bits z and up of 32
      return z >= 32 ? 0u : z <= 0 ? 0xFFFFFFFFu : 0xFFFFFFFFu << z;
    };
    uint32_t bad[T / 2 + 1];                    // 32 accumulators each
#pragma unroll
    for (int k = 0; k < T / 2 + 1; ++k) bad[k] = ~(bits_from(z0 - 32 * k) & ~bits_from(z1 + 1 - 32 * k));
#pragma unroll
    for (int z = 0; z < Z2; ++z) {
      const uint32_t rank = (uint32_t)(RUN - 1 - z % RUN);
      const uint32_t lo = (bad[z / 32] >> (z % 32)) & 1u, hi = (bad[(z + Z2) / 32] >> ((z + Z2) % 32)) & 1u;
      pen[z] = (lo << 15) | (hi << 31) | rank * 0x10001u;
    }
  }
  // every term adds 64 - p . q = 2 popcount(p ^ q) (times 2^(IB - 1)): the windows start at 64
  // per row, above 2^23 so that the low bits of the float are the sum
  v16f acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 8388608.0f + (f_in ? kTerms : 0.0f);
  // rows outside the image read as 0 in both views (no difference), columns outside it as 0
  auto load_row = [&](int y) {
    const bool in = y >= 0 && y < a.H;
    const size_t ro = (size_t)(in ? y : 0) * (size_t)a.pitch;
    const int nrec = in ? W * 8 : 0;
    const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc((void*)(a.CL + ro), (short)0, nrec, 0x00020000);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc((void*)(a.CR + ro), (short)0, nrec, 0x00020000);
    DenseRow<T> w;
    w.f = __builtin_amdgcn_raw_buffer_load_b32(rf, foff, 0, 0);
#pragma unroll
    for (int t = 0; t < T; ++t) w.m[t] = __builtin_amdgcn_raw_buffer_load_b32(rm, moff[t], 0, 0);
    return w;
  };
  auto add_row = [&](const DenseRow<T>& w, uint32_t flip) {
    const v4i f = fp4_signs(w.f ^ flip, fsign, fmag);
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = mfma_fp4(fp4_signs(w.m[t], sign, mag), f, acc[t]);
  };
  const uint32_t cost_bits = in_vgpr(0x10001u * (0xFFFFu & ~(uint32_t)(RUN - 1)));
  const uint32_t lane_rank = 0x10001u * (uint32_t)(n & (RUN - 1));
  uint32_t* __restrict__ put = turn + h * Z2 * DenseTurn<T>::STRIDE + n;
  DenseRow<T> enter = load_row(y0 - R), leave = enter;
#pragma unroll 1
  for (int i = 0; i < NR; ++i) {
    // step i + 1's rows are loaded while step i's sums are reduced
    const DenseRow<T> e = enter, l = leave;
    if (i + 1 < NR) {
      enter = load_row(y0 - R + i + 1);
      if (i + 1 >= NW) leave = load_row(y0 - R + i + 1 - NW);
    }
    add_row(e, 0xFFFFFFFFu);
    if (i >= NW) add_row(l, 0u);
    if (i < 2 * R) continue;
    // P[2R + z]: the sums of accumulators z and z + Z2; below them, those that z = 0's window
    // reaches back to in the upper half (the lower half's first 2R windows do not exist)
    uint32_t P[Z2 + 2 * R];
    auto V = [&](int z) { return __float_as_uint(acc[z / 16][z % 16]); };
    auto pack = [&](int z) { P[2 * R + z] = __builtin_amdgcn_perm(V(z + Z2), V(z < 0 ? 0 : z), 0x05040100u); };
#pragma unroll
    for (int z = -2 * R; z < 0; ++z) pack(z);
    uint32_t key = 0xFFFFFFFFu;
#pragma unroll
    for (int u = 0; u < NRUN; ++u) {
      u16x2 best = {0xFFFF, 0xFFFF};
      // eight windows at a time: their adds are independent, as a DPP operand must not be
      // the result of the instruction just before
#pragma unroll
      for (int z8 = u * RUN; z8 < (u + 1) * RUN && z8 < Z2; z8 += 8) {
        // (packed as they are needed: packed all at once they spilled 25 registers, 177 us)
#pragma unroll
        for (int v = 0; v < 8; ++v) pack(z8 + v);
        uint32_t s[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) s[v] = P[z8 + v];
#pragma unroll
        for (int k = 1; k <= 2 * R; ++k) {
#pragma unroll
          for (int v = 0; v < 8; ++v) s[v] = P[z8 + v + k] + shr1(s[v]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const uint32_t k = s[v] + pen[z8 + v];
          best = __builtin_elementwise_min(best, __builtin_bit_cast(u16x2, k));
          // the right winner of a column is the least over lanes, the same rank for all: the
          // lane's rank in its place (smaller d first)
          put[(z8 + v) * DenseTurn<T>::STRIDE] = and_or(k, cost_bits, lane_rank);
        }
      }
      // widen: cost << 16 | (d - dmin)
      const uint32_t b = __builtin_bit_cast(uint32_t, best);
#pragma unroll
      for (int hw = 0; hw < 2; ++hw) {
        const uint32_t v = hw ? b >> 16 : b & 0xFFFFu;
        const int q = q0 + h * HS + hw * Z2 + u * RUN - R;
        const int base = c - q - (RUN - 1) - a.dlo;
        const uint32_t wide = ((v & ~(uint32_t)(RUN - 1)) << (16 - IB)) + (v & (RUN - 1)) + (uint32_t)base;
        key = min(key, wide);
      }
    }
    uint32_t* kp = keys + (i - 2 * R) * 64 + lane;
    *kp = chunk == 0 ? key : min(*kp, key);
    // right winners: a lane takes a row of the turned keys, RUN columns at a time
    wave_sync();
    const int y = y0 + i - 2 * R;
#pragma unroll
    for (int p = 0; p < (DenseTurn<T>::ROWS + 63) / 64; ++p) {
      const int row = min(lane + 64 * p, DenseTurn<T>::ROWS - 1);
      const bool row_in = DenseTurn<T>::ROWS % 64 == 0 || lane + 64 * p < DenseTurn<T>::ROWS;
      const uint4* __restrict__ in = (const uint4*)(turn + row * DenseTurn<T>::STRIDE);
      u16x2 m[32 / RUN];
#pragma unroll
      for (int g = 0; g < 32 / RUN; ++g) {
        m[g] = u16x2{0xFFFF, 0xFFFF};
#pragma unroll
        for (int j = 0; j < RUN / 4; ++j) {
          const uint4 v = in[g * (RUN / 4) + j];
          m[g] = __builtin_elementwise_min(m[g], __builtin_bit_cast(u16x2, v.x));
          m[g] = __builtin_elementwise_min(m[g], __builtin_bit_cast(u16x2, v.y));
          m[g] = __builtin_elementwise_min(m[g], __builtin_bit_cast(u16x2, v.z));
          m[g] = __builtin_elementwise_min(m[g], __builtin_bit_cast(u16x2, v.w));
        }
      }
      const int hr = row >= Z2 ? 1 : 0, z = row - hr * Z2;
#pragma unroll
      for (int hw = 0; hw < 2; ++hw) {
        const int q = q0 + hr * HS + hw * Z2 + z - R;
        uint32_t rkey = kNoKey;
#pragma unroll
        for (int g = 0; g < 32 / RUN; ++g) {
          const uint32_t b = __builtin_bit_cast(uint32_t, m[g]);
          const uint32_t v = hw ? b >> 16 : b & 0xFFFFu;
          const int base = xs + RUN * g - 2 * R - q - a.dlo;
          rkey = min(rkey, ((v & ~(uint32_t)(RUN - 1)) << (16 - IB)) + (v & (RUN - 1)) + (uint32_t)base);
        }
        if (row_in && rkey < none_from<R>() && q >= 0 && q < W && y < a.H)
          __hip_atomic_fetch_min(a.right + ((size_t)y * W + q), rkey, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    wave_sync();
  }
}

// grid x: waves over the pair's strips and bands, z: pairs
template <int R, int T>
__global__ __launch_bounds__(256, T > 4 ? 2 : 3) void dense_kernel(DenseArgs a) {
  __shared__ uint32_t keys[4 * kBand * 64];
  __shared__ __attribute__((aligned(16))) uint32_t turn[4 * DenseTurn<T>::WORDS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int item = (int)blockIdx.x * 4 + wave;
  const int band = item / a.strips;
  if (band >= a.bands) return;             // whole wave; the kernel has no barrier
  const int y0 = band * kBand, xs = (item % a.strips) * a.cols;
  a.CL += (int64_t)blockIdx.z * a.cl_zstride;
  a.left += (int64_t)blockIdx.z * a.out_zstride;
  a.right += (int64_t)blockIdx.z * a.out_zstride;
  uint32_t* kw = keys + wave * kBand * 64;
#pragma unroll 1
  for (int j = 0; j < a.chunks; ++j)
    dense_chunk<R, T>(a, xs, y0, j, lane, kw, turn + wave * DenseTurn<T>::WORDS);
  const int n = lane & 31, c = xs + n - 2 * R;
#pragma unroll
  for (int o = 0; o < kBand; ++o) {
    // the two lane halves hold different candidates of the same column
    uint32_t key = kw[o * 64 + lane];
    key = min(key, (uint32_t)__shfl_xor((int)key, 32, 64));
    const int y = y0 + o;
    if (lane >= 2 * R && lane < 2 * R + a.cols && c < a.W && y < a.H)
      a.left[(size_t)y * a.W + c] = key >= none_from<R>() ? (int16_t)-1 : (int16_t)(a.d_out + (int)(key & 0xFFFFu));
  }
}

__global__ __launch_bounds__(256) void dense_clear_kernel(uint32_t* p, size_t n) {
  const size_t i = 4 * ((size_t)blockIdx.x * 256 + threadIdx.x);
  if (i + 4 <= n) *(uint4*)(p + i) = uint4{kNoKey, kNoKey, kNoKey, kNoKey};
  else
    for (size_t k = i; k < n; ++k) p[k] = kNoKey;
}

// A call of at most kFew candidates: no room for a chunk of the search, whose products cover 2
// (16 T - 2R) candidate columns whatever the call asks for. The terms are formed on the vector
// ALU instead (two XORs and two popcounts each), one view per launch and a candidate of every
// column per step: a wave takes a strip of 64 - 2R output columns (its lanes: the strip and a
// halo of R columns on each side) and a band of kBand output rows. Pairs of costs share a word
// of two 16-bit halves (at most 49 x 64 = 3136 each); the vertical sums add the entering row
// and drop the one 2R + 1 rows back (a ring in registers), 2R DPP adds finish a window.
//
// Bound: vector ALU. 1920 x 1080, 1 to 8 candidates, both views and the check: 44 / 53 / 59 us
// for R = 1 / 2 / 3, where the products take 73 / 87 / 98 with T = 3 and 59 / 69 / 77 with T = 2
// (960 x 128 of nine offsets, R = 2: 38 against 53 and 43); 9 to 16 candidates would take two
// steps, 70 / 88 / 100 us, and the products no more than they do for one.
constexpr int kFew = 8;
template <int R>
constexpr int few_strip() { return 64 - 2 * R; }

__device__ __forceinline__ uint32_t shl1(uint32_t v) {   // lane i gets lane i + 1
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);
}

// RIGHT = 0: the left view (the term at column x' pairs CL(x') with CR(x' - d)); 1: the right
// view (the term at column x' pairs CL(x' + d) with CR(x'), and is 0 where x' + d is outside).
// MASKED: some lane reads a word outside the image, so every word and term is checked.
// key[o]: output row o's least cost << 8 | (d - dlo).
template <int R, int RIGHT, bool MASKED>
__device__ __forceinline__ void few_rows(const DenseArgs& a, int x, int y0, uint32_t (&key)[kBand]) {
  constexpr int NW = 2 * R + 1, NR = kBand + 2 * R, NP = kFew / 2;
  const int W = a.W;
  // byte offsets of the fixed word and of the moving words within a row (outside the image:
  // column 0, dropped)
  const bool f_in = x >= 0 && x < W;
  const uint32_t f_off = 8u * (uint32_t)(f_in ? x : 0);
  uint32_t m_off[kFew];
  bool m_in[kFew];
#pragma unroll
  for (int j = 0; j < kFew; ++j) {
    const int xm = RIGHT ? x + a.dlo + j : x - a.dlo - j;
    m_in[j] = xm >= 0 && xm < W;
    m_off[j] = 8u * (uint32_t)(m_in[j] ? xm : 0);
  }
  // (an opaque row pitch: the rows' addresses formed one by one, not all held from the start)
  int pitch_bytes = a.pitch * 8;
  asm volatile("" : "+s"(pitch_bytes));
  const char* fixed_img = (const char*)(RIGHT ? a.CR : a.CL);
  const char* moving_img = (const char*)(RIGHT ? a.CL : a.CR);
  uint32_t ring[NW][NP] = {}, V[NP] = {};
  // step i is image row y0 - R + i; rows outside the image read row 0 and are dropped
  auto load_row = [&](int i, uint64_t& f, uint64_t (&mv)[kFew]) {
    const int yy = y0 - R + i;
    const size_t ro = (size_t)(yy >= 0 && yy < a.H ? yy : 0) * (size_t)pitch_bytes;
    f = *(const uint64_t*)(fixed_img + ro + f_off);
#pragma unroll
    for (int j = 0; j < kFew; ++j) mv[j] = *(const uint64_t*)(moving_img + ro + m_off[j]);
  };
  uint64_t f, mv[kFew];
  load_row(0, f, mv);
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    // step i + 1's row is loaded while step i's is summed
    uint64_t nf = 0, nmv[kFew];
    if (i + 1 < NR) load_row(i + 1, nf, nmv);
    const int yy = y0 - R + i;
    uint32_t t[NP] = {};
    if (yy >= 0 && yy < a.H) {
#pragma unroll
      for (int j = 0; j < kFew; ++j) {
        uint32_t c = (uint32_t)__popcll((!MASKED || f_in ? f : 0ull) ^ (!MASKED || m_in[j] ? mv[j] : 0ull));
        if (MASKED && !(RIGHT ? m_in[j] : f_in)) c = 0;
        t[j / 2] |= c << (16 * (j & 1));
      }
    }
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      V[m] += t[m] - ring[i % NW][m];
      ring[i % NW][m] = t[m];
    }
    if (i >= 2 * R) {
      uint32_t best = 0xFFFFFFFFu;
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        uint32_t h = V[m], l = V[m], r = V[m];
#pragma unroll
        for (int k = 0; k < R; ++k) {
          l = shr1(l);
          r = shl1(r);
          h += l + r;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = 2 * m + q;
          const uint32_t k = ((q ? h >> 16 : h & 0xFFFFu) << 8) | (uint32_t)j;
          best = min(best, j < a.nd && (!RIGHT || !MASKED || m_in[j]) ? k : 0xFFFFFFFFu);
        }
      }
      key[i - 2 * R] = best;
    }
    if (i + 1 < NR) {
      f = nf;
#pragma unroll
      for (int j = 0; j < kFew; ++j) mv[j] = nmv[j];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// grid x: strips, y: four bands each, z: pairs. The left view's disparities, or the right view's
// indices (every pixel is written, so that nothing needs to be cleared).
template <int R, int RIGHT>
__global__ __launch_bounds__(256) void dense_few_kernel(DenseArgs a) {
  a.CL += (int64_t)blockIdx.z * a.cl_zstride;
  a.left += (int64_t)blockIdx.z * a.out_zstride;
  a.right += (int64_t)blockIdx.z * a.out_zstride;
  const int lane = threadIdx.x & 63;
  const int band = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int y0 = band * kBand;
  if (y0 >= a.H) return;                   // whole wave; the kernel has no barrier
  const int xw = blockIdx.x * few_strip<R>() - R;   // column of lane 0
  const int x = xw + lane;
  const bool inside = RIGHT ? (xw >= 0 && xw + 63 + a.dlo + kFew - 1 < a.W)
                            : (xw - a.dlo - (kFew - 1) >= 0 && xw + 63 < a.W);
  uint32_t key[kBand];
  if (inside) few_rows<R, RIGHT, false>(a, x, y0, key);
  else few_rows<R, RIGHT, true>(a, x, y0, key);
  if (lane < R || lane >= R + few_strip<R>() || x >= a.W) return;
#pragma unroll
  for (int o = 0; o < kBand; ++o) {
    const int y = y0 + o;
    if (y >= a.H) break;
    if (RIGHT) a.right[(size_t)y * a.W + x] = key[o] == 0xFFFFFFFFu ? kNoKey : key[o] & 0xFFu;
    else a.left[(size_t)y * a.W + x] = (int16_t)(a.d_out + (int)(key[o] & 0xFFu));
  }
}

// The L/R check of one row segment of 256 pixels; disp holds the left winners and receives
// the checked ones. With `right_out` set it receives the right winners' disparities. With
// `partial` set, the workgroup also stores how many of its checked disparities are > d_min at
// partial[(z * H + y) * gridDim.x + blockIdx.x].
__global__ __launch_bounds__(256) void dense_check_kernel(const uint32_t* __restrict__ right, int W, int H,
                                                          int d_out, int lr_tol, int16_t* disp,
                                                          int16_t* __restrict__ right_out, int d_min,
                                                          int32_t* partial) {
  __shared__ int part[4];
  const size_t plane = (size_t)blockIdx.z * W * H;   // pair z of a multi-pair launch
  right += plane;
  disp += plane;
  const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y;
  auto right_disp = [&](int xr) {
    const uint32_t key = right[(size_t)y * W + xr];
    return key == kNoKey ? -1 : (int)(int16_t)(d_out + (int)(key & 0xFFFFu));
  };
  int above = 0;
  if (x < W) {
    const int d = disp[(size_t)y * W + x];
    const int xr = x - d;
    int ok = 0;
    if (d >= 0 && xr >= 0) {
      const int db = right_disp(xr);
      ok = db >= 0 && abs(d - db) <= lr_tol;
    }
    disp[(size_t)y * W + x] = ok ? (int16_t)d : (int16_t)-1;
    if (right_out) right_out[plane + (size_t)y * W + x] = (int16_t)right_disp(x);
    above = ok && d > d_min ? 1 : 0;
  }
  if (!partial) return;   // uniform over the launch
  for (int o = 32; o > 0; o >>= 1) above += __shfl_xor(above, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = above;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[((size_t)blockIdx.z * H + y) * gridDim.x + blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// counts[z] = the sum of map z's n partial counts: one workgroup per map, no atomics
__global__ __launch_bounds__(256) void count_above_kernel(const int32_t* __restrict__ partial, int n,
                                                          int32_t* counts) {
  __shared__ int part[4];
  const int32_t* p = partial + (size_t)blockIdx.x * n;
  int c = 0;
  for (int i = threadIdx.x; i < n; i += 256) c += p[i];
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Both views' winners of nz pairs in one launch. A wave covers chunks x 2 (16 T - 2R)
// candidate columns for at most 32 - 2R output columns; the shape (T, chunks, columns) with
// the least work per output column is taken (a chunk's work: T products and reductions and
// about 0.9 of one for the fixed column, the right winners and the row's overhead, fitted to
// T = 3, 4 and 5 each alone at 48 to 256 candidates, where the shape taken is within 3% of the
// best of them). T = 2 is for short searches: 1920 x 1080, R = 2, 9 to 28 candidates 69 us, 32
// 75, 36 83, against 87 with T = 3, which is taken from 40 on.
template <int R>
hipError_t launch_dense_r(DenseArgs a, hipStream_t s, int nz) {
  if (a.nd <= kFew) {
    const dim3 grid((a.W + few_strip<R>() - 1) / few_strip<R>(), (a.H + 4 * kBand - 1) / (4 * kBand), nz);
    dense_few_kernel<R, 0><<<grid, 256, 0, s>>>(a);
    dense_few_kernel<R, 1><<<grid, 256, 0, s>>>(a);
    return hipGetLastError();
  }
  int best_t = 0;
  double best = 0;
  for (int t = 2; t <= 5; ++t) {
    const int per = 2 * (16 * t - 2 * R);
    for (int n = (a.nd + 7 + per - 1) / per; n <= (a.nd + 31) / per + 1; ++n) {
      const int cols = std::min(32 - 2 * R, n * per - a.nd + 1);
      const double work = n * (t + 0.9) / cols;
      if (cols >= 8 && (best_t == 0 || work < best)) {
        best = work;
        best_t = t;
        a.cols = cols;
        a.chunks = n;
      }
    }
  }
  const size_t words = (size_t)nz * a.W * a.H;
  dense_clear_kernel<<<(unsigned)((words + 1023) / 1024), 256, 0, s>>>(a.right, words);
  a.strips = (a.W + a.cols - 1) / a.cols;
  a.bands = (a.H + kBand - 1) / kBand;
  const dim3 grid((a.strips * a.bands + 3) / 4, 1, nz);
  if (best_t == 2) dense_kernel<R, 2><<<grid, 256, 0, s>>>(a);
  else if (best_t == 3) dense_kernel<R, 3><<<grid, 256, 0, s>>>(a);
  else if (best_t == 4) dense_kernel<R, 4><<<grid, 256, 0, s>>>(a);
  else dense_kernel<R, 5><<<grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_dense_any(const DenseArgs& a, int radius, hipStream_t s, int nz) {
  if (radius == 1) return launch_dense_r<1>(a, s, nz);
  if (radius == 2) return launch_dense_r<2>(a, s, nz);
  if (radius == 3) return launch_dense_r<3>(a, s, nz);
  return hipErrorNotSupported;
}

}  // namespace

bool dense_radius_supported(int radius) { return radius >= 1 && radius <= 3; }

hipError_t launch_dense(const uint64_t* CL, const uint64_t* CR, int W, int H, int pitch, int dmin,
                        int dmax, int radius, int lr_tol, int16_t* disp, uint32_t* right,
                        int16_t* disp_right, hipStream_t stream, const LaunchTimer* timer) {
  const DenseArgs args = {CL, CR, W, H, pitch, std::min(dmin, W + 512), dmax - dmin + 1, dmin, disp, right,
                          0, 0, 0, 0, 0, 0};
  if (timer) timer->before(timer->ctx, "dense", stream);
  const hipError_t e = launch_dense_any(args, radius, stream, 1);
  if (timer) timer->after(timer->ctx, "dense", stream);
  if (e != hipSuccess) return e;
  if (timer) timer->before(timer->ctx, "dense_check", stream);
  dense_check_kernel<<<dim3((W + 255) / 256, H), 256, 0, stream>>>(right, W, H, dmin, lr_tol, disp,
                                                                   disp_right, 0, nullptr);
  if (timer) timer->after(timer->ctx, "dense_check", stream);
  return hipGetLastError();
}

// Dense counterpart of nz pairs at once: pair z is (CL0 - z rows, CR), i.e. the left
// descriptors moved down by z more rows; then the pixels above d_min of each map.
hipError_t launch_dense_offsets(const uint64_t* CL0, const uint64_t* CR, int W, int H, int pitch,
                                int nz, int dmin, int dmax, int radius, int lr_tol, int d_min,
                                int16_t* disp, uint32_t* right, int32_t* partial, int32_t* counts,
                                hipStream_t stream, const LaunchTimer* timer) {
  const DenseArgs args = {CL0, CR, W, H, pitch, std::min(dmin, W + 512), dmax - dmin + 1, dmin, disp, right,
                          -(int64_t)pitch, (int64_t)W * H, 0, 0, 0, 0};
  if (timer) timer->before(timer->ctx, "rect_dense", stream);
  const hipError_t e = launch_dense_any(args, radius, stream, nz);
  if (timer) timer->after(timer->ctx, "rect_dense", stream);
  if (e != hipSuccess) return e;
  if (timer) timer->before(timer->ctx, "rect_count", stream);
  const int bx = (W + 255) / 256;
  dense_check_kernel<<<dim3(bx, H, nz), 256, 0, stream>>>(right, W, H, dmin, lr_tol, disp, nullptr, d_min,
                                                          partial);
  count_above_kernel<<<nz, 256, 0, stream>>>(partial, H * bx, counts);
  if (timer) timer->after(timer->ctx, "rect_count", stream);
  return hipGetLastError();
}

}  // namespace ocsr
