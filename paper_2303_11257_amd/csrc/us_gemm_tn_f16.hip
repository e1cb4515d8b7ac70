// GEMM family: grad_W product dW = X^T G: both operands K-strided (the reduction runs over tokens),
// cut into K slices with an ordered FP32 reduction when the output alone cannot fill the chip.
#include "us_gemm_dispatch.h"

namespace us {

hipError_t gemm_tn_f16(const GemmProblem& p, hipStream_t st) {
  const int splits = p.workspace && small_tile_choice(p) == SmallTileChoice::None ? gemm_splits(p.M, p.N, p.K) : 1;
  if (splits <= 1) return launch_store<false, 0, 0, false, false>(p, st);
  const long k_per_split = gemm_k_per_split(p.K, splits);
  hipError_t e = launch_sized<false, 0, 0, false, false, EPI_PARTIAL, true>(p, splits, k_per_split, st);
  if (e != hipSuccess) return e;
  return launch_splitk_reduce((const float*)p.workspace, p.C, p.M * p.N, splits, p.scale, p.c_dt == US_F32, st);
}

// Two equally shaped FP16 batches in one launch.  Results of up to 64 columns take 256-row tiles where they pad no more rows than
// 128-row tiles and still make two per CU, else 128-row tiles (forward + backward of attention back to back, us, 128 x 128 / 128 x 64 / 256 x
// 64 tiles: 256 heads x 512 x 64 275 / 275 / 267, 512 x 192 x 64 97 / 95 / 90, 400 x 384 x 64 272 / 265 / 274, 16 x 2048 x 64
// 423 / 410 / 446, 1024 x 128 x 64 84.3 / 82.3 / 83.7; one launch instead of two: 64 x 128 x 64
// 21.8 -> 18.0, 128 x 512 x 128 215 -> 202).  128 x 128 tiles of up to two stages in the form for short reductions: 1024 x 64 x 80 49.2 -> 48.9, 1024 x 32 x 128 41.7 -> 41.3
// (300 x 144 x 80 even, 256 x 192 x 128 81.6 -> 80.2 without).
hipError_t gemm_tn_f16_two_batches(const GemmProblem& p, const GemmProblem& q, hipStream_t st) {
  if (!offsets_fit(p)) return hipErrorInvalidValue;
  if (p.N > 64) return 2 * p.K <= CfgD128::NST * CfgD128::BKB ? launch_two_batches<Short<CfgD128>>(p, q, st) : launch_two_batches<CfgD128>(p, q, st);
  const long t128 = ceil_div(p.M, 128), t256 = ceil_div(p.M, 256);
  if (2 * t256 <= t128 && 2 * p.batch * t256 >= 2 * cu_count()) return launch_two_batches<CfgN256>(p, q, st);
  return launch_two_batches<CfgN128>(p, q, st);
}

}  // namespace us
