// Matching with a vertical range (the census cost over (dx, dy), Sec. 4.3.2): the matrix-core
// matchers, each direction repeated for every vertical offset.
#include <algorithm>

#include "match_kernels.hpp"

namespace ocsr {
namespace {

template <int CPL>
using VPair = dev::MatrixMatcher<2, CPL, true>;
template <int CPL>
using VQuad = dev::MatrixMatcher<4, CPL, true>;

// Waves per SIMD: those of matrix_waves, but four 4 x 4 blocks per wave hold half the digits
template <int ROWS, int CPL>
constexpr int v_waves() { return ROWS == 2 ? matrix_waves<CPL>() : CPL <= 2 ? 4 : CPL <= 8 ? 3 : 2; }

hipError_t launch_level(const MatchParamsDev& P, const FramesDev& FR, const MatchWs& ws,
                        const DebugDev& dbg, int level, int grid, hipStream_t stream,
                        const LaunchTimer* timer) {
  const PathDev& v = P.path[level];
  const bool want = dbg.blocks || dbg.cost_fwd || dbg.cost_bwd;
#define OCSR_V(ROWS, M, C)                                                                     \
  if (v.rows == ROWS && v.cpl == C)                                                            \
    return timed_launch(timer, "match",                                                       \
                        want ? match_level_kernel<M<C>, v_waves<ROWS, C>(), true>             \
                             : match_level_kernel<M<C>, v_waves<ROWS, C>(), false>,           \
                        dim3(grid), dim3(256), 0, stream, P, FR, ws, dbg, level);
  OCSR_V(1, VQuad, 2)
  OCSR_V(1, VQuad, 4)
  OCSR_V(1, VQuad, 8)
  OCSR_V(1, VQuad, 12)
  OCSR_V(1, VQuad, 16)
  OCSR_V(2, VPair, 1)
  OCSR_V(2, VPair, 2)
  OCSR_V(2, VPair, 3)
  OCSR_V(2, VPair, 4)
  OCSR_V(2, VPair, 5)
#undef OCSR_V
  return hipErrorNotSupported;   // rejected by the argument checks before any launch
}

}  // namespace

hipError_t launch_match_vertical(const MatchParamsDev& P, const FramesDev& FR, const MatchWs& ws,
                                 const DebugDev& dbg, int grid, int level_launches,
                                 hipStream_t stream, const LaunchTimer* timer) {
  const PathDev& f = P.path[0];
  const PathDev& c = P.path[1];
  if (level_launches != 1 && !dbg.blocks && !dbg.cost_fwd && !dbg.cost_bwd) {
    // Both levels in one launch: the far blocks run beside the close ones. A level of few blocks
    // takes as long as one group's walk over the offsets, so that a launch each adds the two up:
    // 1080p, 32 boxes, dy -1..1, far and close 8 x 8, us with one launch and with two: 35 and 45
    // over 64 candidates, 39 and 51 over 96, 42 and 62 over 128.
#define OCSR_VP(FM, FROWS, FROM, FCPL, CM, CROWS, CCPL)                                       \
    if (f.rows == FROWS && f.cpl >= FROM && f.cpl <= FCPL && c.rows == CROWS && c.cpl == CCPL) \
      return timed_launch(timer, "match",                                                     \
                          match_pair2_kernel<FM<FCPL>, CM<CCPL>,                              \
                                             std::min(v_waves<FROWS, FCPL>(), v_waves<CROWS, CCPL>())>, \
                          dim3(grid), dim3(256), 0, stream, P, FR, ws);
#define OCSR_VP5(FM, FROWS, FCPL)                                                             \
    OCSR_VP(FM, FROWS, FCPL, FCPL, VPair, 2, 1)                                               \
    OCSR_VP(FM, FROWS, FCPL, FCPL, VPair, 2, 2)                                               \
    OCSR_VP(FM, FROWS, FCPL, FCPL, VPair, 2, 3)                                               \
    OCSR_VP(FM, FROWS, FCPL, FCPL, VPair, 2, 4)                                               \
    OCSR_VP(FM, FROWS, FCPL, FCPL, VPair, 2, 5)
    OCSR_VP5(VQuad, 1, 2)
    OCSR_VP5(VQuad, 1, 8)
    OCSR_VP5(VQuad, 1, 12)
    OCSR_VP5(VQuad, 1, 16)
    OCSR_VP5(VPair, 2, 1)
    OCSR_VP5(VPair, 2, 2)
    OCSR_VP5(VPair, 2, 3)
    OCSR_VP5(VPair, 2, 4)
    OCSR_VP5(VPair, 2, 5)
#define OCSR_VP_QUAD(CCPL)                                                                    \
    OCSR_VP(VQuad, 1, 2, 2, VQuad, 1, CCPL)                                                   \
    OCSR_VP(VQuad, 1, 4, 8, VQuad, 1, CCPL)                                                   \
    OCSR_VP(VQuad, 1, 12, 16, VQuad, 1, CCPL)                                                 \
    OCSR_VP(VPair, 2, 1, 2, VQuad, 1, CCPL)                                                   \
    OCSR_VP(VPair, 2, 3, 5, VQuad, 1, CCPL)
    OCSR_VP_QUAD(8)
    OCSR_VP_QUAD(12)
    OCSR_VP_QUAD(16)
#undef OCSR_VP_QUAD
#undef OCSR_VP5
#undef OCSR_VP
  }
  for (int level = 1; level >= 0; --level) {
    const hipError_t e = launch_level(P, FR, ws, dbg, level, grid, stream, timer);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ocsr
