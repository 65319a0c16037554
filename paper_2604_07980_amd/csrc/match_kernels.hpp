// Matching kernels over any matcher, shared by the translation units that launch them.
#pragma once

#include "dev_matrix.hpp"

namespace ocsr {
namespace {

// Both levels in one launch with any pair of matchers (FM far, CM close): work items of
// every frame's close level first, then of every far level. Compiled for WAVES waves per
// SIMD. (Calls with debug output take one launch per level.)
template <class FM, class CM, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES))) void match_pair2_kernel(
    MatchParamsDev P, FramesDev FR, MatchWs ws) {
  const DebugDev dbg = {};
  constexpr size_t kWave = FM::kLds > CM::kLds ? FM::kLds : CM::kLds;
  __shared__ uint64_t lds[(kItemWaves * kWave + 7) / 8];
  __shared__ int prefix[2 * kMaxFrames + 1];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int F = FR.n;
  if (threadIdx.x < 64) {
    const int j = lane < F ? lane : lane - F;
    const int cnt = lane < 2 * F ? ws.fcount[j * FC_N + (lane < F ? FC_CLOSE_ITEMS : FC_FAR_ITEMS)] : 0;
    const int incl = dev::wave_incl_scan(cnt);
    if (lane < 2 * F) prefix[lane + 1] = incl;
    if (lane == 0) prefix[0] = 0;
  }
  __syncthreads();
  void* wl = (char*)lds + wave * kWave;
  // the close items of every frame, then the far ones, dealt XCD by XCD as two lists
  const int n_close = prefix[F], n_all = prefix[2 * F];
  const int sh = dev::share_items(n_all, FM::kShares && CM::kShares ? P.share_groups : 0);
  const dev::Deal2 dl = dev::xcd_deal2(n_close << sh, (n_all - n_close) << sh);
  for (int i = dl.first; i < dl.end; i += dl.step) {
    const int at = dl.at(i), m = at >> sh;
    const int sub = sh ? at & (kItemWaves - 1) : -1;
    int slot = 0;
    for (int k = 1; k < 2 * F; ++k)
      if (m >= prefix[k]) slot = k;
    const int f = slot < F ? slot : slot - F;
    const FrameDev& fr = FR.f[f];
    const int q = m - prefix[slot];
    // the lane index passes through an empty asm statement per item, so that neither
    // matcher's per-lane indexing is held in registers across the loop (both would be)
    int il = lane;
    asm volatile("" : "+v"(il));
    if (slot < F) {
      const typename CM::State st = CM::frame_state(ws, fr, il);
      ItemRec r = dev::find_item(P, fr, FR.n_boxes_total, ws, 1, q, il);
      r.sub = sub;
      CM::run_item(P, fr, ws, dbg, f, 1, r, wave, il, wl, st);
    } else {
      const typename FM::State st = FM::frame_state(ws, fr, il);
      ItemRec r = dev::find_item(P, fr, FR.n_boxes_total, ws, 0, q, il);
      r.sub = sub;
      FM::run_item(P, fr, ws, dbg, f, 0, r, wave, il, wl, st);
    }
  }
}

// Waves per SIMD the matrix-core matchers are compiled for: their strip and accumulators grow
// with the candidates per lane, and as many waves are taken as leave few registers to spill in
// the built code. Four candidates per lane would spill 8 at four waves: a 2160p frame of 200 boxes
// takes 91.3 us instead of 92.8, 16 x 1200p of 40 boxes over 128 level candidates 118 instead of
// 123 (blocks of one point, with little to spill, 443 instead of 422). With a vertical range they
// would spill 50: a 1080p frame of 32 + 32 boxes over dy -3..3 takes 60 us instead of 66, a 2160p
// one of 120 boxes 210 instead of 238. (Three candidates, spilling 11, measure 49.5 instead of
// 51.3 on the first but 161 instead of 158 on the second, and stay at four waves. Both with a
// wave walking all offsets of its group.)
template <int CPL>
constexpr int matrix_waves() { return CPL <= 3 ? 4 : CPL <= 6 ? 3 : 2; }

// One level with any matcher. Without DBG no debug output is asked for, and its code and
// pointers are not in the kernel.
template <class M, int WAVES, bool DBG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES))) void match_level_kernel(
    MatchParamsDev P, FramesDev FR, MatchWs ws, DebugDev dbg_, int level) {
  const DebugDev dbg = DBG ? dbg_ : DebugDev{};
  __shared__ uint64_t lds[(kItemWaves * M::kLds + 7) / 8];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  void* wl = (char*)lds + wave * M::kLds;
  dev::level_items(FR, ws, level, M::kShares && !DBG ? P.share_groups : 0, [&](int f, int q, int sub) {
    const FrameDev& fr = FR.f[f];
    const typename M::State st = M::frame_state(ws, fr, lane);
    ItemRec r = dev::find_item(P, fr, FR.n_boxes_total, ws, level, q, lane);
    r.sub = sub;
    M::run_item(P, fr, ws, dbg, f, level, r, wave, lane, wl, st);
  });
}

}  // namespace
}  // namespace ocsr
