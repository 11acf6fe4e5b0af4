// Row-statistics pass of the score kernels (pass 1): per query row, the
// maximum and the sum of exp(s - max) over one column block.
#include "score.h"
#include "score_wave.h"

namespace catekv {

hipError_t launch_score_rowstats(int dtype, int G, bool causal, int rows_pad, dim3 grid, hipStream_t s,
                                 const ScoreArgs& a) {
  if (dtype == CATEKV_BF16) {
    if (score_wave_rows(rows_pad)) return launch_score_wave<kRowStats>(grid, s, a);
#define CATEKV_SC(GG, CC) \
  if ((GG == 0 || G == GG) && causal == CC) { \
    hipLaunchKernelGGL((score_kernel<uint16_t, 16, 2, kRowStats, GG, CC, 4>), grid, dim3(1024), 0, s, a); \
    return hipGetLastError(); \
  }
    CATEKV_SC(0, false) CATEKV_SC(1, true) CATEKV_SC(2, true) CATEKV_SC(4, true) CATEKV_SC(8, true)
#undef CATEKV_SC
    return hipErrorInvalidValue;
  }
  // without a mask the group size only places Q rows: one build
  if (!causal) return launch_score_mt<float, kRowStats, 0, false>(rows_pad, grid, s, a);
#define CATEKV_SC(GG) \
  if (G == GG) return launch_score_mt<float, kRowStats, GG, true>(rows_pad, grid, s, a);
  CATEKV_SC(1) CATEKV_SC(2) CATEKV_SC(4) CATEKV_SC(8)
#undef CATEKV_SC
  return hipErrorInvalidValue;
}

}  // namespace catekv
