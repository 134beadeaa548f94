// launch.hpp -- host-side launchers of the gfx950 kernels (library-internal).
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"

namespace gt4mi {

// Longest column the fused (register-resident) column kernels accept.
constexpr int kMaxFusedNk = 160;

// fused forward (k_step.hip dispatches; k_step_inst.hip instantiates the
// register classes of each dtype / tile / column store)
template <typename T>
hipError_t launch_step_fused(StepArgs<T> A, int tile_i, int tile_j, int column_store, hipStream_t s);
template <typename T, int TI, int TJ, int COL>
hipError_t launch_step_classes(const StepArgs<T>& A, hipStream_t s);
template <typename T, int COL>
hipError_t launch_vadv_classes(const StepArgs<T>& A, hipStream_t s);
// VAR: the generalised diffusion (per-point coefficient, damping form)
template <typename T, int TI, int TJ, bool VAR>
hipError_t launch_split_classes(const StepArgs<T>& A, hipStream_t s);
// FP64 columns of 97..144 levels in 128-column tiles (k_split.hpp)
template <typename T, int TI>
hipError_t launch_split_long(const StepArgs<T>& A, hipStream_t s);
// two-ended column solve: ADJ = false, out = T^{-1}(u + data);
// ADJ = true, out = T^{-T} u (u holds x_bar); nk <= 144 (FP64) / 160 (FP32)
template <typename T, bool ADJ>
hipError_t launch_column_split_classes(StepArgs<T> A, hipStream_t s);
constexpr int column_split_limit(int elem_bytes) { return elem_bytes == 8 ? 144 : 160; }
// Columns per tile of the two-ended fused step (two lanes per column) in one
// compilation of k_step_inst.hip: 256 makes 512-lane workgroups, 128 makes
// 256-lane ones; both are built and the tile option (a tuned dimension)
// picks one.
#ifndef GT4MI_SPLIT_NT
#define GT4MI_SPLIT_NT 256
#endif
// two-ended fused step (k_split.hpp): nk <= 144 (FP64) / 160 (FP32)
constexpr int split_step_limit(int elem_bytes) { return elem_bytes == 8 ? 144 : 160; }
constexpr int kCus = 256;  // of the chip
// Workgroups of its 256-column tiles that a CU holds: each has two waves per SIMD, of
// the 4, 3, 2, 2, 2 (FP64: up to 32, 48, 80, 96, 144 levels) and 7, 5, 4, 3, 2 (FP32:
// 32, 48, 80, 112, 160) that the registers of the class in k_split.hpp leave.
constexpr int split_tiles_per_cu(int elem_bytes, int64_t nk) {
  return elem_bytes == 8 ? (nk <= 32 ? 2 : 1) : nk <= 32 ? 3 : nk <= 80 ? 2 : 1;
}
template <typename T>
hipError_t launch_vadv_fused(StepArgs<T> A, hipStream_t s);
template <typename T>
hipError_t launch_hdiff_fused(StepArgs<T> A, int tile_i, hipStream_t s);

// plain per-stage forward (k_plain.hip); ws holds the stage temporaries
template <typename T>
struct PlainWs {
  T* lap;  // (ni+2) x (nj+2) x nk
  T* fx;   // (ni+1) x nj x nk
  T* fy;   // ni x (nj+1) x nk
  T* cp;   // ni x nj x nk
  T* dp;   // ni x nj x nk
};
template <typename T>
hipError_t launch_hdiff_plain(const StepArgs<T>& A, const PlainWs<T>& ws, hipStream_t s);
// out = T^{-1}(u + data) with u, data, out given by A; elimination factors in ws
template <typename T>
hipError_t launch_vadv_plain(const StepArgs<T>& A, const PlainWs<T>& ws, hipStream_t s);

// adjoints (k_adjoint.hip; column classes in k_vadj_inst.hip)
template <typename T>
hipError_t launch_vadv_adjoint(AdjArgs<T> A, int impl_plain, T* ws_y, T* ws_c, hipStream_t s);
template <typename T, int COL>
hipError_t launch_vadj_classes(const AdjArgs<T>& A, hipStream_t s);
template <typename T>
hipError_t launch_hdiff_adjoint(AdjArgs<T> A, hipStream_t s);

// batched launches (k_batched.hip).  The work list sits in device memory: a
// BatchHeader, then prefix[n + 1] (first work item of each field), then the
// fields' argument blocks, fields sorted longest column first.
struct BatchHeader {
  int32_t n;      // fields
  int32_t total;  // work items
  int32_t pad[2];
  __host__ __device__ const int32_t* prefix() const { return reinterpret_cast<const int32_t*>(this + 1); }
};
// The part of a table that one launch runs: n consecutive fields, whose
// first items are at prefix (a device pointer) and whose work items are
// first .. first + items - 1.
struct BatchRange {
  const int32_t* prefix;
  int32_t n, first, items;
};
// longest column of a batched field
constexpr int kMaxBatchedNk = 144;
// stream-ordered copy of a small host table into device memory (kernel
// arguments, so that a captured graph holds its own copy)
hipError_t launch_upload(void* dst, const void* src, size_t bytes, hipStream_t s);

// Register classes of the batched forward step, longest columns first: the
// fields of a class share one launch.  max_nk: its longest column; nkh: levels
// of a half column held in VGPRs; nt: columns per tile; pd: levels loaded ahead.
// Each argument block names its field's tile width (StepArgs::tile_i).
constexpr int kStepBatchClasses = 3;
template <typename T, int C>
struct StepBatchClass;
template <>
struct StepBatchClass<double, 0> {
  static constexpr int max_nk = 144, nkh = 72, nt = kSplitLongNT, pd = 4;
};
template <>
struct StepBatchClass<double, 1> {
  static constexpr int max_nk = 96, nkh = 48, nt = 256, pd = 2;
};
template <>
struct StepBatchClass<double, 2> {
  static constexpr int max_nk = 80, nkh = 40, nt = 256, pd = 2;
};
template <>
struct StepBatchClass<float, 0> {
  static constexpr int max_nk = 144, nkh = 72, nt = 128, pd = 2;
};
template <>
struct StepBatchClass<float, 1> {
  static constexpr int max_nk = 112, nkh = 56, nt = 128, pd = 2;
};
template <>
struct StepBatchClass<float, 2> {
  static constexpr int max_nk = 80, nkh = 40, nt = 256, pd = 2;
};
// class of a column, and the columns per tile of a class
template <typename T>
constexpr int step_batch_class(int64_t nk) {
  return nk <= StepBatchClass<T, 2>::max_nk ? 2 : nk <= StepBatchClass<T, 1>::max_nk ? 1 : 0;
}
template <typename T>
constexpr int step_batch_nt(int cls) {
  return cls == 0 ? StepBatchClass<T, 0>::nt : cls == 1 ? StepBatchClass<T, 1>::nt : StepBatchClass<T, 2>::nt;
}
template <typename T>
hipError_t launch_step_batched(int cls, const BatchRange& r, const StepArgs<T>* ent, bool mask, hipStream_t s);

// column adjoint: class 0 above kVadjBatchedShortNk levels, class 1 up to it;
// the rows of its 64-wide tiles
constexpr int kVadjBatchedShortNk = 96;
int vadj_batched_tile_rows(bool f64, int cls);
template <typename T>
hipError_t launch_vadj_batched(int cls, const BatchRange& r, const StepArgs<T>* ent, hipStream_t s);
template <typename T>
hipError_t launch_hadj_batched(const BatchRange& r, const AdjArgs<T>* ent, hipStream_t s);

// parameter gradients of a step (k_param.hip)
template <typename T>
struct WGradArgs {
  const T* w;  // staggered level 0 at domain (0,0)
  int64_t w_sj, w_sk;
  const T* x;  // the step's output
  int64_t x_sj, x_sk;
  const T* lam;  // T^{-T} x_bar
  int64_t l_sj, l_sk;
  T* wbar;  // staggered, nk+1 levels written
  int64_t b_sj, b_sk;
  int ni, nj, nk, tiles_i;
  T q;  // dt_dz / 4
};
// Partial sums of the coeff gradient (doubles): the fewest the launch takes, one
// per 64 x 4 tile, and the most it uses, one per strip workgroup and level.
inline int64_t coeff_partial_least(int64_t ni, int64_t nj) { return ((ni + 63) / 64) * ((nj + 3) / 4); }
int64_t coeff_partial_most(bool f64, int64_t ni, int64_t nj, int64_t nk);
// A: u (halo) and lam in the data slot; W may be NULL (no w_bar); coeff_bar may
// be NULL (no reduction; partial unused), a float if f32; slots: doubles at partial
template <typename T>
hipError_t launch_param_grads(const StepArgs<T>& A, const WGradArgs<T>* W, double* partial, int64_t slots,
                              void* coeff_bar, bool f32, hipStream_t s);

// gradient of a per-point coefficient: A.out(p) = -A.data(p) D(u)(p)
// (A.data holds lam; A.form selects the Laplacian form)
template <typename T>
hipError_t launch_coeff_field_grad(const StepArgs<T>& A, hipStream_t s);

// periodic halo fill of a padded field (p at domain (0,0,0); k_halo.hip)
template <typename T>
hipError_t launch_halo_periodic(T* p, int64_t sj, int64_t sk, int ni, int nj, int nk, hipStream_t s);

// the same for two fields of one domain
template <typename T>
hipError_t launch_halo_periodic_pair(T* p, int64_t p_sj, int64_t p_sk, T* q, int64_t q_sj, int64_t q_sk, int ni, int nj,
                                     int nk, hipStream_t s);

// fill a strided box with a deterministic pattern (autotuner scratch)
template <typename T>
hipError_t launch_fill_pattern(T* p, int64_t n, T lo, T hi, uint32_t seed, hipStream_t s);

}  // namespace gt4mi
