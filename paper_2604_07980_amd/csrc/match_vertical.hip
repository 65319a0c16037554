// Matching with a vertical range (the census cost over (dx, dy), Sec. 4.3.2): the matrix-core
// matchers, each direction repeated for every vertical offset.
#include "match_kernels.hpp"

namespace ocsr {
namespace {

template <int CPL>
using VPair = dev::MatrixMatcher<2, CPL, true>;
template <int CPL>
using VQuad = dev::MatrixMatcher<4, CPL, true>;

hipError_t launch_level(const MatchParamsDev& P, const FramesDev& FR, const MatchWs& ws,
                        const DebugDev& dbg, int level, int grid, hipStream_t stream,
                        const LaunchTimer* timer) {
  const PathDev& v = P.path[level];
  const bool want = dbg.blocks || dbg.cost_fwd || dbg.cost_bwd;
#define OCSR_V(ROWS, M, C)                                                                     \
  if (v.rows == ROWS && v.cpl == C)                                                            \
    return timed_launch(timer, "match",                                                       \
                        want ? match_level_kernel<M<C>, matrix_waves<C, true>(), true>        \
                             : match_level_kernel<M<C>, matrix_waves<C, true>(), false>,      \
                        dim3(grid), dim3(256), 0, stream, P, FR, ws, dbg, level);
  OCSR_V(1, VQuad, 2)
  OCSR_V(1, VQuad, 4)
  OCSR_V(2, VPair, 1)
  OCSR_V(2, VPair, 2)
  OCSR_V(2, VPair, 3)
  OCSR_V(2, VPair, 4)
  OCSR_V(2, VPair, 5)
  OCSR_V(2, VPair, 6)
  OCSR_V(2, VPair, 8)
#undef OCSR_V
  return hipErrorNotSupported;   // rejected by the argument checks before any launch
}

}  // namespace

hipError_t launch_match_vertical(const MatchParamsDev& P, const FramesDev& FR, const MatchWs& ws,
                                 const DebugDev& dbg, int grid, int level_launches,
                                 hipStream_t stream, const LaunchTimer* timer) {
  const PathDev& f = P.path[0];
  const PathDev& c = P.path[1];
  if (level_launches != 1 && !dbg.blocks && !dbg.cost_fwd && !dbg.cost_bwd && f.rows == 1 && f.cpl == 2 && c.rows == 2) {
    // both levels in one launch for the usual pairs: the far blocks run beside the close ones
#define OCSR_VP(C)                                                                            \
    if (c.cpl == C)                                                                           \
      return timed_launch(timer, "match", match_pair2_kernel<VQuad<2>, VPair<C>, matrix_waves<C, true>()>, \
                          dim3(grid), dim3(256), 0, stream, P, FR, ws);
    OCSR_VP(2)
    OCSR_VP(3)
    OCSR_VP(4)
    OCSR_VP(5)
#undef OCSR_VP
  }
  for (int level = 1; level >= 0; --level) {
    const hipError_t e = launch_level(P, FR, ws, dbg, level, grid, stream, timer);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ocsr
