// k_hdiff.hip -- launcher of the horizontal diffusion alone: the row walk
// (k_hdiff_strip.hpp), or the tile kernel (k_step.hpp) where that is faster
// (by_tiles), where the walk's 32-bit mask window does not reach and, for the
// generalised diffusion, beyond kMaxGridY levels (the stated form walks those too:
// tested with 65543).
#include "k_hdiff_strip.hpp"
#include "k_step.hpp"

namespace gt4mi {

// Whether 32 x 8 tiles are faster than the walk.
// Narrow domains: strips (56 columns, FP32 two to a lane 120) span 1.3 times the
// columns of tiles or more.  Walk and tiles, us, stated FP64 / damping FP64 / damping
// FP32, by the ratio: 62x700x100 (1.75, FP32 1.88) 18.9 15.7 / 23.4 17.3 / 14.1 12.5;
// 121x119x140 (1.31, 1.88) 9.7 8.9 / 11.4 10.2 / 9.6 8.1; 72x530x105 (1.17, 1.25)
// 15.5 17.0 / 19.3 19.6 / 11.8 13.9; 200x200x60 (1, 1.07) 9.0 10.3 / 10.5 11.7 / 8.4
// 9.0.
// With a mask, whose bits the walk stores byte by byte, all domains of up to 2^22
// points.  Walk and tiles, stated / kappa field, on cold buffers: FP32 384x384x20
// 11.2 10.1 / 12.2 11.2, 450x150x60 13.4 12.6 / 15.1 14.1, 384x384x64 21.4 24.1 /
// 29.5 33.3; FP64 384x384x20 12.6 12.2 / 15.2 13.9, 450x150x60 17.1 16.3 / 23.7 23.5,
// 384x384x64 36.1 41.2 / 49.6 51.9.
template <typename T>
static bool by_tiles(const StepArgs<T>& A) {
  constexpr int64_t w = sizeof(T) == 4 ? kHStripOut2 : kHStripOut;
  const int64_t strips = (A.ni + w - 1) / w * w, tiles = (A.ni + 31) / 32 * 32;
  if (A.nj > 1 << 26) return false;  // a grid counts its lanes in 32 bits
  return 10 * strips >= 13 * tiles || (A.mask && (int64_t)A.ni * A.nj * A.nk <= 1 << 22);
}

template <typename T>
hipError_t launch_hdiff_fused(StepArgs<T> A, int tile_i, hipStream_t s) {
  const bool var = A.kappa != nullptr || A.form != 0;  // the generalised diffusion
  // the walk addresses the mask through one 32-bit window
  const bool small_mask = A.mask == nullptr || A.ml.total <= (int64_t)kOffNone - 16;
  if (small_mask && by_tiles(A)) {
    tile_i = 32;
  } else if (small_mask) {
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
