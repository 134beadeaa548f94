// k_hdiff.hip -- launcher of the horizontal diffusion alone: the row walk
// (k_hdiff_strip.hpp), or the tile kernel (k_step.hpp) where the walk's 32-bit
// mask window does not reach and, for the generalised diffusion, beyond kMaxGridY
// levels (the stated form has walked those from the first and runs on every nk:
// tested with 65543).
#include "k_hdiff_strip.hpp"
#include "k_step.hpp"

namespace gt4mi {

template <typename T>
hipError_t launch_hdiff_fused(StepArgs<T> A, int tile_i, hipStream_t s) {
  const bool var = A.kappa != nullptr || A.form != 0;  // the generalised diffusion
  // the walk addresses the mask through one 32-bit window
  const bool small_mask = A.mask == nullptr || A.ml.total <= (int64_t)kOffNone - 16;
  if (small_mask) {
    // strips of 56 columns (FP32: 120, two columns per lane), four per workgroup,
    // one level per grid row (the tile option does not apply)
    if (!var) return launch_hdiff_strip<T, kHPlain>(A, s);
    if (A.nk <= kMaxGridY) return launch_hdiff_strip<T, kHVar>(A, s);
  }
  // a tile marched over a block of levels; enough workgroups to fill the chip
  const int tj = kWG / tile_i;
  A.tiles_i = (A.ni + tile_i - 1) / tile_i;
  A.ntiles = A.tiles_i * ((A.nj + tj - 1) / tj);
  int kper = A.nk;
  while (kper > 4 && (int64_t)A.ntiles * ((A.nk + kper - 1) / kper) < 4096) kper = (kper + 1) / 2;
  A.k1 = kper;
  dim3 grid(A.ntiles, (A.nk + kper - 1) / kper), block(kWG);
#define GT4MI_HDIFF_LAUNCH(TI, TJ)                                                  \
  if (var)                                                                          \
    hipLaunchKernelGGL((k_hdiff_fused<T, TI, TJ, true>), grid, block, 0, s, A);    \
  else                                                                              \
    hipLaunchKernelGGL((k_hdiff_fused<T, TI, TJ, false>), grid, block, 0, s, A);
  if (tile_i == 64) {
    GT4MI_HDIFF_LAUNCH(64, 4)
  } else if (tile_i == 32) {
    GT4MI_HDIFF_LAUNCH(32, 8)
  } else {
    GT4MI_HDIFF_LAUNCH(16, 16)
  }
#undef GT4MI_HDIFF_LAUNCH
  return hipGetLastError();
}

template hipError_t launch_hdiff_fused<float>(StepArgs<float>, int, hipStream_t);
template hipError_t launch_hdiff_fused<double>(StepArgs<double>, int, hipStream_t);

}  // namespace gt4mi
