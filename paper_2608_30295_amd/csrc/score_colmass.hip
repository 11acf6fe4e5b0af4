// Column-mass pass of the score kernels (pass 2 of the selection): the
// group-mean attention mass of every key column, or with a chunk size that
// divides the 64-column tile its chunk maxima (BlockMax) directly.
#include "score.h"
#include "score_wave.h"

namespace catekv {

hipError_t launch_score_colmass(int dtype, bool wave, int rows_pad, dim3 grid, hipStream_t s, const ScoreArgs& a) {
  if (wave) return launch_score_wave<kColMass>(grid, s, a);
  return dtype == CATEKV_BF16 ? launch_score_mt<uint16_t, kColMass, 0, false>(rows_pad, grid, s, a)
                              : launch_score_mt<float, kColMass, 0, false>(rows_pad, grid, s, a);
}

// A few heads' samples leave compute units idle: their rows are split there
// (one head, 256 rows: 8.4 -> 4.9 us).
hipError_t launch_score_est(int n_sel, hipStream_t s, const ScoreArgs& a) {
  const int rg = sw_row_tiles(a.R), fit = 8 / n_sel;   // 32 workgroups per head, 256 compute units
  const int split = fit >= 8 ? 8 : fit >= 4 ? 4 : fit >= 2 ? 2 : 1;
  return launch_score_wave<kRowEst>(dim3(kSwEstParts, n_sel, std::min(split, rg)), s, a);
}
hipError_t launch_score_both(dim3 grid, hipStream_t s, const ScoreArgs& a) { return launch_score_wave<kBoth>(grid, s, a); }
hipError_t launch_score_gather(dim3 grid, hipStream_t s, const ScoreArgs& a) {
  return launch_score_wave<kColGather>(grid, s, a);
}

}  // namespace catekv
