// k_hdiff.hip -- launcher of the horizontal diffusion alone: the row walk
// (k_hdiff_strip.hpp), or the tile kernel (k_step.hpp) where that is faster
// (by_tiles), where the walk's 32-bit mask window does not reach and, for the
// generalised diffusion, beyond kMaxGridY levels (the stated form walks those too:
// tested with 65543).
#include "k_hdiff_strip.hpp"
#include "k_step.hpp"

namespace gt4mi {

// Whether 32 x 8 tiles are faster than the walk; us, walk and tiles, the fields in the
// last-level cache / on cold buffers.
// Narrow domains, by the columns that strips (56, FP32 two to a lane 120) and tiles
// span, their ratio: FP64 1.75 64x900x140 stated 30.6 27.3 / 32.9 34.2, with the mask
// 41.9 29.7 / 42.9 37.6, damping 38.4 29.6 / 45.0 35.6; 1.31 128x512x120 24.0 26.8 /
// 29.4 35.4, 31.5 28.8 / 33.3 35.8, 29.0 29.2 / 36.1 34.9, but in few points (121x119x140)
// 9.7 8.9, 12.4 10.1, 11.4 10.2; 1.17 72x530x105 15.5 17.0, 20.8 18.9, 19.3 19.6.  FP32
// 1.88 122x600x100 stated 15.5 16.6 / 15.6 17.4, with the mask 24.6 18.7 / 24.6 18.6,
// damping 20.9 18.3 / 20.8 18.2; 1.41 256x512x80 18.1 21.1 / 19.6 27.0, 24.7 23.1 / 26.6
// 30.5, 20.9 23.5 / 24.8 27.8; 3.75 22x897x61 stated 9.7 6.1, damping 11.4 7.0.
// With a mask, whose bits the walk stores byte by byte, all domains of up to 2^22
// points: stated / kappa field on cold buffers, FP32 384x384x20 11.2 10.1 / 12.2 11.2,
// 450x150x60 13.4 12.6 / 15.1 14.1, 384x384x64 21.4 24.1 / 29.5 33.3; FP64 384x384x20
// 12.6 12.2 / 15.2 13.9, 450x150x60 17.1 16.3 / 23.7 23.5, 384x384x64 36.1 41.2 / 49.6
// 51.9.
template <typename T>
static bool by_tiles(const StepArgs<T>& A, bool var) {
  constexpr int64_t w = sizeof(T) == 4 ? kHStripOut2 : kHStripOut;
  const int64_t strips = (A.ni + w - 1) / w * w, tiles = (A.ni + 31) / 32 * 32;
  const bool few = (int64_t)A.ni * A.nj * A.nk <= 1 << 22;
  if (A.nj > 1 << 26) return false;  // a grid counts its lanes in 32 bits
  if (reinterpret_cast<uintptr_t>(A.mask) % 4) return false;  // tiles store whole words of it
  if (A.mask && few) return true;
  const int tenths = sizeof(T) == 8 ? (few ? 13 : 15) : var || A.mask ? 15 : 30;
  return 10 * strips >= tenths * tiles;
}

template <typename T>
hipError_t launch_hdiff_fused(StepArgs<T> A, int tile_i, hipStream_t s) {
  const bool var = A.kappa != nullptr || A.form != 0;  // the generalised diffusion
  // the walk addresses the mask through one 32-bit window
  const bool small_mask = A.mask == nullptr || A.ml.total <= (int64_t)kOffNone - 16;
  if (small_mask && by_tiles(A, var)) {
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
