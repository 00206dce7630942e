// Declarations of the staged covariance smoother (smooth_staged.hip) for its
// callers: the covariance smoother and batched cross-validation.
#pragma once

#include <vector>

#include "common.hpp"

namespace fpca {

// One fit: C = Ca - Cb and G = Ga - Gb (Cb, Gb may be null; Ca null: c0 off the
// diagonal). Cross-validation scores it against the held-out fold's slabs.
struct StagedJob {
  const void *Ca, *Cb, *Ga, *Gb;
  const void *Qf, *Gf, *Cf;
  double c0;
  const double *h;  // d bandwidths
};

// d = 2 and 3, P <= 4096 and at most 40 nodes per coordinate.
bool staged_supported(const fpca_grid *grid);
// Whether the handle's covariance fits on this grid are staged ones: the default
// engine, and direct moment sums (the other convolution modes ask for the pass
// engine's FFT, which the staged kernels have no place for).
inline bool takes_staged(const fpca_context *ctx, const fpca_grid *grid) {
  return ctx->engine == FPCA_ENGINE_AUTO && ctx->conv_mode == FPCA_CONV_DIRECT && staged_supported(grid);
}
// b0 of one fit at every node (and its status, optional).
template <typename T>
int staged_smooth(fpca_context *ctx, const fpca_grid *grid, const StagedJob &job, T *out, int8_t *status);
// The scores of the jobs, to `scores` (device, one per job).
template <typename T>
int staged_scores(fpca_context *ctx, const fpca_grid *grid, const std::vector<StagedJob> &jobs, double *scores);

}  // namespace fpca
