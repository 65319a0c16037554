// Multi-launch path (Alg. 2): census and plan of every frame in one launch, one
// matching launch per level, one aggregation launch. A matching launch deals work items
// (up to item_blocks blocks of one box, spread over the four waves of a workgroup)
// over its grid; the aggregation launch gives each box a workgroup that forms its
// disparity (Sec. 4.3.4) and depth (Eq. 1). Results cross workgroups only at kernel
// boundaries. The device steps are in dev_census.hpp and dev_match.hpp, shared with
// the fused persistent kernel.
#include "dev_census.hpp"
#include "match_kernels.hpp"

namespace ocsr {
namespace {

// one wave per frame (descriptor-level calls, whose census is the caller's)
__global__ __launch_bounds__(64) void plan_kernel(MatchParamsDev P, FramesDev FR,
                                                  const ocsr_box* boxes, MatchWs ws) {
  const int f = blockIdx.x;
  dev::plan_frame(P, FR.f[f], f, FR.n_boxes_total, boxes, ws, threadIdx.x);
}

// workgroups 0 .. n_frames - 1 plan a frame each (one wave); the rest make the census, one
// tile each (a workgroup tests whether some box's search reads its tile)
template <int SX, int SY>
__global__ __launch_bounds__(256) void frame_census_kernel(MatchParamsDev P, FramesDev FR,
                                                           const ocsr_box* boxes, MatchWs ws,
                                                           int sx, int sy, int sentinel) {
  __shared__ alignas(dev::kCensusLdsAlign) uint32_t lds[SX >= 0 ? dev::CensusTile<(SX > 0 ? SX : 0), (SY > 0 ? SY : 0)>::kLdsBytes / 4 : 1];
  __shared__ int tsc[4];
  if ((int)blockIdx.x < FR.n) {
    if (threadIdx.x < 64)
      dev::plan_frame(P, FR.f[blockIdx.x], blockIdx.x, FR.n_boxes_total, boxes, ws, threadIdx.x);
    return;
  }
  dev::frame_census_tile<SX, SY>(P, FR, boxes, blockIdx.x - FR.n, sx, sy, sentinel, lds, true,
                                 &tsc[0]);
}

// Plan of frame blockIdx.x and the list of its census tiles. Wave 0 plans the boxes while
// waves 1-3 mark the tiles their searches read, each wave in a tile map of its own (so
// the marking waits for no workgroup barrier, and the plan and the marking overlap);
// then all four waves list the tiles of the three maps.
__global__ __launch_bounds__(256) void plan_tiles_kernel(MatchParamsDev P, FramesDev FR,
                                                         const ocsr_box* boxes, MatchWs ws) {
  constexpr int kMaps = kItemWaves - 1;
  __shared__ uint32_t bits[kMaps * kFrameTileWords];
  __shared__ int sc[8];
  const int f = blockIdx.x;
  const FrameDev& fr = FR.f[f];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  if (wave == 0) {
    dev::plan_frame(P, fr, f, FR.n_boxes_total, boxes, ws, lane);
  } else {
    uint32_t* map = bits + (wave - 1) * kFrameTileWords;
    const int n_tiles = 2 * (fr.tiles0 + fr.tiles1);
    const int n_words = (n_tiles + 31) >> 5;
    for (int i = lane; i < n_words; i += 64) map[i] = dev::tile_map_init(P, n_tiles, i);
    dev::wave_sync();
    if (!P.full_census) dev::mark_frame_tiles(P, fr, boxes, map, (int)threadIdx.x - 64, 192);
  }
  __syncthreads();
  dev::compact_frame_tiles(fr, f, ws, bits, kMaps, kFrameTileWords, sc);
}

// Census of the listed tiles of every frame by persistent workgroups: the frames' lists,
// concatenated, are shared out in equal consecutive parts, the parts of one XCD's
// workgroups adjacent (neighbouring tiles read overlapping source rows).
template <int SX, int SY>
__global__ __launch_bounds__(256) void census_list_kernel(MatchParamsDev P, FramesDev FR,
                                                          const ocsr_box* boxes, MatchWs ws,
                                                          int sx, int sy, int sentinel) {
  __shared__ alignas(dev::kCensusLdsAlign) uint32_t lds[SX >= 0 ? dev::CensusTile<(SX > 0 ? SX : 0), (SY > 0 ? SY : 0)>::kLdsBytes / 4 : 1];
  __shared__ int pre[kMaxFrames + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < 64) {
    const int cnt = lane < FR.n ? ws.fcount[lane * FC_N + FC_TILES] : 0;
    const int incl = dev::wave_incl_scan(cnt);
    if (lane < FR.n) pre[lane + 1] = incl;
    if (lane == 0) pre[0] = 0;
  }
  __syncthreads();
  const int N = pre[FR.n];
  const int G = gridDim.x, b = blockIdx.x, x = b & 7;
  int w = 0;   // this workgroup's rank when the workgroups of XCD 0 come first, then XCD 1, ...
  for (int y = 0; y < x; ++y) w += (G - y + 7) >> 3;
  w += b >> 3;
  const int lo = dev::share_start(N, w, G), hi = dev::share_start(N, w + 1, G);
  int f = 0;
  auto job = [&](int q) {
    while (q >= pre[f + 1]) ++f;
    const FrameDev& fr = FR.f[f];
    return dev::frame_tile_local(fr, f, fr.tile_list[q - pre[f]]).job;
  };
  for (int q = lo; q < hi; ++q) {
    dev::make_census_tile<SX, SY>(job(q), sx, sy, sentinel, lds);
    __syncthreads();   // the next tile reuses the LDS
  }
}

// Waves per SIMD a single-level kernel is compiled for (as many as its registers allow
// without spilling, checked in the built code).
template <int ROWS, int CPL, int PASSES>
constexpr int tiled_waves() {
  return ROWS == 4 ? ((CPL <= 2 || (CPL <= 4 && PASSES == 1)) ? 6 : CPL <= 8 ? 4 : 2)
                   : (CPL <= 4 && PASSES == 1) ? 5
                   : ((CPL <= 4 && PASSES <= 3) || (CPL <= 6 && PASSES <= 2)) ? 4
                   : CPL <= 12 ? 3 : CPL <= 16 ? 2 : 1;
}

template <int ROWS, int NX, int CPL, int PASSES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(tiled_waves<ROWS, CPL, PASSES>()))) void match_tiled_kernel(MatchParamsDev P, FramesDev FR,
                                                          MatchWs ws, DebugDev dbg, int level) {
  constexpr size_t kWave = (dev::Tiled<ROWS, NX, CPL, PASSES>::kLdsBytes + 15) & ~(size_t)15;
  __shared__ uint64_t lds[(kItemWaves * kWave + 7) / 8];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  void* wl = (char*)lds + wave * kWave;
  dev::level_items(FR, ws, level, 0, [&](int f, int q, int) {
    const FrameDev& fr = FR.f[f];
    const ItemRec r = dev::find_item(P, fr, FR.n_boxes_total, ws, level, q, lane);
    dev::run_item_rec(P, fr, f, level, r, wave, [&](const dev::BlockCtx& c) {
      dev::match_block_tiled<ROWS, NX, CPL, PASSES>(P, fr, ws, dbg, c, lane, wl);
    });
  });
}

// Waves per SIMD the paired kernel is compiled for: three where both variants fit in a
// third of the register file without spilling (checked in the built code), else two.
template <int FR_, int FC, int CC, int CP>
constexpr int pair_waves() {
  return CP > 1 ? (CC <= 6 ? 4 : 3)
         : ((FR_ == 4 && FC <= 2 && CC <= 12) || (FC <= 8 && CC <= 8)) ? 3 : 2;
}

// Both levels in one launch: work items of every frame's close level first, then of
// every far level (FV / CV: the far and close kernel variants).
template <int FR_, int FX, int FC, int CR_, int CX, int CC, int CP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pair_waves<FR_, FC, CC, CP>()))) void match_pair_kernel(MatchParamsDev P, FramesDev FR,
                                                         MatchWs ws) {
  const DebugDev dbg = {};
  constexpr size_t kF = (dev::Tiled<FR_, FX, FC>::kLdsBytes + 15) & ~(size_t)15;
  constexpr size_t kC = (dev::Tiled<CR_, CX, CC, CP>::kLdsBytes + 15) & ~(size_t)15;
  constexpr size_t kWave = kF > kC ? kF : kC;
  __shared__ uint64_t lds[(kItemWaves * kWave + 7) / 8];
  __shared__ int prefix[2 * kMaxFrames + 1];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int F = FR.n;
  if (threadIdx.x < 64) {
    // prefix[j]: items before slot j; slot j < F is frame j's close level, else frame
    // j - F's far level
    const int j = lane < F ? lane : lane - F;
    const int cnt = lane < 2 * F ? ws.fcount[j * FC_N + (lane < F ? FC_CLOSE_ITEMS : FC_FAR_ITEMS)] : 0;
    const int incl = dev::wave_incl_scan(cnt);
    if (lane < 2 * F) prefix[lane + 1] = incl;
    if (lane == 0) prefix[0] = 0;
  }
  __syncthreads();
  void* wl = (char*)lds + wave * kWave;
  const int n_close = prefix[F];
  const dev::Deal2 dl = dev::xcd_deal2(n_close, prefix[2 * F] - n_close);
  for (int i = dl.first; i < dl.end; i += dl.step) {
    const int m = dl.at(i);
    int slot = 0;
    for (int k = 1; k < 2 * F; ++k)
      if (m >= prefix[k]) slot = k;
    const int f = slot < F ? slot : slot - F;
    const FrameDev& fr = FR.f[f];
    const int q = m - prefix[slot];
    const ItemRec r = dev::find_item(P, fr, FR.n_boxes_total, ws, slot < F ? 1 : 0, q, lane);
    if (slot < F) {
      dev::run_item_rec(P, fr, f, 1, r, wave, [&](const dev::BlockCtx& c) {
        dev::match_block_tiled<CR_, CX, CC, CP>(P, fr, ws, dbg, c, lane, wl);
      });
    } else {
      dev::run_item_rec(P, fr, f, 0, r, wave, [&](const dev::BlockCtx& c) {
        dev::match_block_tiled<FR_, FX, FC>(P, fr, ws, dbg, c, lane, wl);
      });
    }
  }
}

__global__ __launch_bounds__(256) void aggregate_kernel(MatchParamsDev P, MatchWs ws,
                                                        ocsr_box_result* out) {
  __shared__ dev::AggLds sm;
  dev::aggregate_box(P, ws, blockIdx.x, out, false, sm);
}

}  // namespace

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

size_t match_ws_bytes(int n_frames, int n_boxes_total, int cap_blocks) {
  const size_t n = (size_t)(n_boxes_total > 0 ? n_boxes_total : 1);
  const size_t c = (size_t)(cap_blocks > 0 ? cap_blocks : 1) * (size_t)(n_frames > 0 ? n_frames : 1);
  return align256(n * sizeof(BoxPlan)) + align256(n * sizeof(BoxClip)) +
         align256(2 * n * sizeof(int32_t)) +
         align256((size_t)kMaxFrames * FC_N * sizeof(int32_t)) + align256(GC_N * sizeof(int32_t)) +
         2 * align256(c * sizeof(float)) + align256(c * sizeof(uint8_t)) +
         (size_t)(n_frames > 0 ? n_frames : 1) * reserved_bytes(n_boxes_total, cap_blocks);
}

MatchWs match_ws_carve(void* base, int n_frames, int n_boxes_total, int cap_blocks) {
  const size_t n = (size_t)(n_boxes_total > 0 ? n_boxes_total : 1);
  const size_t c = (size_t)(cap_blocks > 0 ? cap_blocks : 1) * (size_t)(n_frames > 0 ? n_frames : 1);
  char* b = (char*)base;
  MatchWs ws;
  ws.plan = (BoxPlan*)b;        b += align256(n * sizeof(BoxPlan));
  ws.clip = (BoxClip*)b;        b += align256(n * sizeof(BoxClip));
  ws.litem_end = (int32_t*)b;   b += align256(2 * n * sizeof(int32_t));
  ws.fcount = (int32_t*)b;      b += align256((size_t)kMaxFrames * FC_N * sizeof(int32_t));
  ws.gcount = (int32_t*)b;      b += align256(GC_N * sizeof(int32_t));
  ws.blk_val = (float*)b;       b += align256(c * sizeof(float));
  ws.agg_tmp = (float*)b;       b += align256(c * sizeof(float));
  ws.blk_flag = (uint8_t*)b;    b += align256(c * sizeof(uint8_t));
  return ws;
}

namespace {
// the built kernels, as in launch_level, in order of preference for the default
struct BuiltVariant { int rows, nx, cpl, passes; };
// rows = 2: two blocks of up to 8 x 8 points per wave on the matrix cores, cpl candidates on
// each of 32 lanes; rows = 1: four blocks of up to 4 x 4, cpl candidates on each of 16 lanes
constexpr BuiltVariant kBuilt[] = {
    {1, 4, 2, 1},  {1, 4, 4, 1},
    {4, 4, 2, 1},  {2, 8, 1, 1},  {2, 8, 2, 1},  {2, 8, 3, 1},  {2, 8, 4, 1},  {2, 8, 5, 1},
    {2, 8, 6, 1},  {2, 8, 8, 1},
    {4, 4, 4, 1},  {4, 4, 8, 1},  {4, 4, 16, 1}, {8, 8, 4, 1},  {8, 8, 8, 1},
    {8, 8, 6, 2},  {8, 8, 12, 1}, {8, 8, 16, 1}, {8, 8, 24, 1}, {8, 8, 32, 1}, {8, 8, 4, 2},
    {8, 8, 4, 3},  {8, 8, 4, 4},  {8, 8, 8, 2},  {4, 4, 2, 2},  {4, 4, 4, 2},
    {0, 8, 4, 1}};
}  // namespace

bool variant_valid(const PathDev& ph, int rows, int cpl, int passes) {
  // rows = 0: the generic kernel, any TILED block of up to 64 points or a GRID block
  if (rows == 0 && cpl == 4 && passes == 1)
    return ph.nd <= 256 && (ph.mode == OCSR_MODE_GRID ? ph.n_side <= 8 : ph.bw * ph.bh <= 64);
  if (ph.mode != OCSR_MODE_TILED) return false;
  for (const BuiltVariant& b : kBuilt)
    if (b.rows == rows && b.cpl == cpl && b.passes == passes)
      return b.rows == 0   ? false
             : b.rows == 1 ? ph.bw <= 4 && ph.bh <= 4 && 16 * b.cpl >= ph.nd
             : b.rows == 2 ? ph.bw <= 8 && ph.bh <= 8 && 32 * b.cpl >= ph.nd
                           : ph.bw <= b.nx && ph.bh <= b.rows && (64 / b.rows) * b.cpl * b.passes >= ph.nd;
  return false;
}

int variant_candidates(const PathDev& ph, int* rows, int* cpl, int* passes, int cap) {
  int n = 0;
  for (const BuiltVariant& b : kBuilt) {
    if (!variant_valid(ph, b.rows, b.cpl, b.passes)) continue;
    if (n < cap) {
      rows[n] = b.rows;
      cpl[n] = b.cpl;
      passes[n] = b.passes;
    }
    ++n;
  }
  return n;
}

MatchVariant pick_variant(const PathDev& ph) {
  for (const BuiltVariant& b : kBuilt)
    if (variant_valid(ph, b.rows, b.cpl, b.passes)) return MatchVariant{1, b.rows, b.cpl, b.passes};
  return MatchVariant{0, 0, 0, 0};
}

static hipError_t launch_level(const MatchParamsDev& P, const FramesDev& FR, const MatchWs& ws,
                               const DebugDev& dbg, int level, int grid, hipStream_t stream,
                               const LaunchTimer* timer, const char* name) {
  const PathDev& v = P.path[level];
#define OCSR_TILED(R, X, C, PS)                                                             \
  if (v.rows == R && v.cpl == C && v.passes == PS)                                          \
    return timed_launch(timer, name, match_tiled_kernel<R, X, C, PS>, dim3(grid), dim3(256), 0, \
                        stream, P, FR, ws, dbg, level);
  OCSR_TILED(4, 4, 2, 1)
  OCSR_TILED(4, 4, 4, 1)
  OCSR_TILED(4, 4, 8, 1)
  OCSR_TILED(4, 4, 16, 1)
  OCSR_TILED(8, 8, 4, 1)
  OCSR_TILED(8, 8, 8, 1)
  OCSR_TILED(8, 8, 12, 1)
  OCSR_TILED(8, 8, 16, 1)
  OCSR_TILED(8, 8, 24, 1)
  OCSR_TILED(8, 8, 32, 1)
  OCSR_TILED(8, 8, 4, 2)
  OCSR_TILED(8, 8, 4, 3)
  OCSR_TILED(8, 8, 4, 4)
  OCSR_TILED(8, 8, 6, 2)
  OCSR_TILED(8, 8, 8, 2)
  OCSR_TILED(4, 4, 2, 2)
  OCSR_TILED(4, 4, 4, 2)
#undef OCSR_TILED
  const bool want = dbg.blocks || dbg.cost_fwd || dbg.cost_bwd;
#define OCSR_LEVEL(M, WAVES)                                                                  \
  return timed_launch(timer, name, want ? match_level_kernel<M, WAVES, true> : match_level_kernel<M, WAVES, false>, \
                      dim3(grid), dim3(256), 0, stream, P, FR, ws, dbg, level)
#define OCSR_TWO(C)                                                                           \
  if (v.rows == 2 && v.cpl == C) OCSR_LEVEL(dev::PairMatcher<C>, matrix_waves<C>())
  OCSR_TWO(1);
  OCSR_TWO(2);
  OCSR_TWO(3);
  OCSR_TWO(4);
  OCSR_TWO(5);
  OCSR_TWO(6);
  OCSR_TWO(8);
#undef OCSR_TWO
  if (v.rows == 0) OCSR_LEVEL(dev::GenericMatcher, 4);
  if (v.rows == 1 && v.cpl == 2) OCSR_LEVEL(dev::QuadMatcher<2>, 4);
  if (v.rows == 1 && v.cpl == 4) OCSR_LEVEL(dev::QuadMatcher<4>, 4);
#undef OCSR_LEVEL
  return hipErrorNotSupported;   // rejected by the argument checks before any launch
}

// One launch for both levels when a kernel for the pair of variants is built (with
// launch == false: only whether it is built).
#define COMMA ,
static bool launch_pair(const MatchParamsDev& P, const FramesDev& FR, const MatchWs& ws, int grid, hipStream_t stream, const LaunchTimer* timer,
                        bool launch) {
  const PathDev& f = P.path[0];
  const PathDev& c = P.path[1];
  if (f.passes != 1) return false;
#define OCSR_PAIR(FRW, FXW, FCP, CRW, CXW, CCP, CPS)                                     \
  if (f.rows == FRW && f.cpl == FCP && c.rows == CRW && c.cpl == CCP && c.passes == CPS) { \
    if (launch)                                                                          \
      timed_launch(timer, "match", match_pair_kernel<FRW, FXW, FCP, CRW, CXW, CCP, CPS>,    \
                   dim3(grid), dim3(256), 0, stream, P, FR, ws);                          \
    return true;                                                                         \
  }
  OCSR_PAIR(4, 4, 2, 8, 8, 8, 1)
  OCSR_PAIR(4, 4, 2, 8, 8, 12, 1)
  OCSR_PAIR(4, 4, 2, 8, 8, 16, 1)
  OCSR_PAIR(4, 4, 4, 8, 8, 8, 1)
  OCSR_PAIR(4, 4, 4, 8, 8, 12, 1)
  OCSR_PAIR(8, 8, 8, 8, 8, 8, 1)
  OCSR_PAIR(8, 8, 8, 8, 8, 12, 1)
  OCSR_PAIR(8, 8, 8, 8, 8, 16, 1)
  OCSR_PAIR(4, 4, 2, 8, 8, 4, 3)
  OCSR_PAIR(4, 4, 2, 8, 8, 6, 2)
  OCSR_PAIR(4, 4, 2, 8, 8, 4, 2)
#undef OCSR_PAIR
#define OCSR_PAIR2(FM, FRW, FCP, FPS, CCP)                                                  \
  if (f.rows == FRW && f.cpl == FCP && f.passes == FPS && c.rows == 2 && c.cpl == CCP) {    \
    if (launch)                                                                          \
      timed_launch(timer, "match", match_pair2_kernel<FM, dev::PairMatcher<CCP>, matrix_waves<CCP>()>, dim3(grid),  \
                   dim3(256), 0, stream, P, FR, ws);                                      \
    return true;                                                                         \
  }
  OCSR_PAIR2(dev::TiledMatcher<4 COMMA 4 COMMA 2 COMMA 1>, 4, 2, 1, 2)
  OCSR_PAIR2(dev::TiledMatcher<4 COMMA 4 COMMA 2 COMMA 1>, 4, 2, 1, 3)
  OCSR_PAIR2(dev::TiledMatcher<4 COMMA 4 COMMA 2 COMMA 1>, 4, 2, 1, 4)
  OCSR_PAIR2(dev::PairMatcher<1>, 2, 1, 1, 3)
  OCSR_PAIR2(dev::PairMatcher<2>, 2, 2, 1, 3)
  OCSR_PAIR2(dev::PairMatcher<2>, 2, 2, 1, 4)
  OCSR_PAIR2(dev::PairMatcher<3>, 2, 3, 1, 3)
  OCSR_PAIR2(dev::QuadMatcher<2>, 1, 2, 1, 2)
  OCSR_PAIR2(dev::QuadMatcher<2>, 1, 2, 1, 5)
  OCSR_PAIR2(dev::QuadMatcher<2>, 1, 2, 1, 6)
  OCSR_PAIR2(dev::QuadMatcher<2>, 1, 2, 1, 8)
  OCSR_PAIR2(dev::QuadMatcher<2>, 1, 2, 1, 3)
  OCSR_PAIR2(dev::QuadMatcher<2>, 1, 2, 1, 4)
  OCSR_PAIR2(dev::GenericMatcher, 0, 4, 1, 3)
#undef OCSR_PAIR2
  return false;
}

hipError_t launch_frame_census(const MatchParamsDev& P, const FramesDev& FR,
                               const ocsr_box* boxes, const MatchWs& ws, int sx, int sy,
                               int sentinel, int n_census_tiles, hipStream_t stream,
                               const LaunchTimer* timer) {
  const dim3 grid(FR.n + n_census_tiles), block(256);
  auto kernel = sx == 3 && sy == 4   ? frame_census_kernel<3, 4>
                : sx == 2 && sy == 2 ? frame_census_kernel<2, 2>
                : sx == 4 && sy == 3 ? frame_census_kernel<4, 3>
                                     : frame_census_kernel<-1, -1>;
  return timed_launch(timer, "census", kernel, grid, block, 0, stream, P, FR, boxes, ws, sx, sy,
                      sentinel);
}

template <int SX, int SY>
static int census_list_occupancy() {
  static const int occ = [] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, census_list_kernel<SX, SY>, 256, 0) != hipSuccess)
      n = 1;
    return n > 0 ? n : 1;
  }();
  return occ;
}

hipError_t launch_plan_and_census(const MatchParamsDev& P, const FramesDev& FR,
                                  const ocsr_box* boxes, const MatchWs& ws, int sx, int sy,
                                  int sentinel, int n_cu, hipStream_t stream,
                                  const LaunchTimer* timer) {
  int n_tiles = 0;
  for (int f = 0; f < FR.n; ++f) {
    const int t = 2 * (FR.f[f].tiles0 + FR.f[f].tiles1);
    if (t > 32 * kFrameTileWords) return hipErrorNotSupported;
    n_tiles += t;
  }
  const bool w34 = sx == 3 && sy == 4, w22 = sx == 2 && sy == 2, w43 = sx == 4 && sy == 3;
  const int occ = w34 ? census_list_occupancy<3, 4>() : w22 ? census_list_occupancy<2, 2>()
                  : w43 ? census_list_occupancy<4, 3>() : census_list_occupancy<-1, -1>();
  // lists pay off once every persistent workgroup has several tiles to consider, and sooner
  // with many frames, as a frame's list is one workgroup's work. Whole calls, listed against
  // one workgroup per tile, us: one 2160p frame (10200 tiles) 56.2 and 51.5, two (20400) 82.4
  // and 87.6; 2 x 1200p (5700) 39.6 and 36.6, 4 (11400) 45.8 and 47.8, 6 (17100) 60.6 and 66.4;
  // 8 x 720p (9280) 31.1 and 34.9, 8 x 600p (5840) 32.4 and 33.0
  const int per_slot = FR.n >= 8 ? 3 : FR.n >= 4 ? 5 : 8;
  if (per_slot * std::max(1, n_cu) * occ > n_tiles) return hipErrorNotSupported;
  hipError_t e = timed_launch(timer, "plan", plan_tiles_kernel, dim3(FR.n), dim3(256), 0, stream, P,
                              FR, boxes, ws);
  if (e != hipSuccess) return e;
  auto kernel = w34 ? census_list_kernel<3, 4> : w22 ? census_list_kernel<2, 2>
                : w43 ? census_list_kernel<4, 3> : census_list_kernel<-1, -1>;
  // (shares are cut in 32-bit arithmetic, which takes grids below 46341)
  return timed_launch(timer, "census", kernel, dim3(std::min(std::max(1, n_cu) * occ, 46340)), dim3(256), 0, stream,
                      P, FR, boxes, ws, sx, sy, sentinel);
}

double match_work(const FramesDev& FR) {
  double work = 0;
  for (int f = 0; f < FR.n; ++f) work += (double)FR.f[f].n_boxes * FR.f[f].W * FR.f[f].H;
  return work;
}

hipError_t launch_match(const MatchParamsDev& P, const FramesDev& FR, const ocsr_box* boxes,
                        const MatchWs& ws, ocsr_box_result* out, const DebugDev& dbg,
                        bool plan_done, int n_match_wgs, int level_launches, hipStream_t stream,
                        const LaunchTimer* timer) {
  if (FR.n_boxes_total <= 0) return hipSuccess;
  hipError_t e;
  if (!plan_done) {
    if (timer) timer->before(timer->ctx, "plan", stream);
    plan_kernel<<<FR.n, 64, 0, stream>>>(P, FR, boxes, ws);
    if (timer) timer->after(timer->ctx, "plan", stream);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (P.vertical) {
    e = launch_match_vertical(P, FR, ws, dbg, n_match_wgs, level_launches, stream, timer);
    if (e != hipSuccess) return e;
  } else if (!dbg.blocks && !dbg.cost_fwd && !dbg.cost_bwd &&
             (level_launches == 2 ||
              (level_launches == 0 &&
               (FR.n == 1 || match_work(FR) < (P.item_blocks[1] > kItemWaves ? 2000e6 : 700e6)))) &&
             launch_pair(P, FR, ws, n_match_wgs, stream, nullptr, false)) {
    // one launch for both levels: the far level alone cannot fill the GPU, and its blocks
    // fill the close level's tail. Whole calls, one launch against two: 1080p frame 24.9 and
    // 30.6 us, 3 x 717p 23.5 and 29.0, 8 x 1200p 74.0 and 77.7, 16 x 1200p 115.9 and 118.2.
    // The kernel of both levels has more registers to spill, and past a batch of that size
    // one launch per level is no slower: 16 x 1200p of 1088 boxes 171.9 us against 174.3 (within
    // what one call differs by between processes); with items of one group per wave from
    // 8 x 1200p on (79.7 against 79.8, 123.0 against 130.5)
    e = launch_pair(P, FR, ws, n_match_wgs, stream, timer, true) ? hipGetLastError() : hipErrorNotSupported;
    if (e != hipSuccess) return e;
  } else {
    // close blocks first: they carry most of the work
    for (int level = 1; level >= 0; --level) {
      e = launch_level(P, FR, ws, dbg, level, n_match_wgs, stream, timer,
                       level == 0 ? "match_far" : "match_close");
      if (e != hipSuccess) return e;
    }
  }
  return timed_launch(timer, "aggregate", aggregate_kernel, dim3(FR.n_boxes_total), dim3(256), 0,
                      stream, P, ws, out);
}

}  // namespace ocsr
