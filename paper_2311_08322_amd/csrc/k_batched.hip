// k_batched.hip -- kernels that run a batch of fields of uneven sizes in a
// few launches, one per register class of the column length.
//
// The host sorts the fields longest column first and writes a table into
// the caller's workspace (a header with the per-field prefix sums of work
// items, then one argument block per field) with small copy kernels, so the
// whole call is stream-ordered device work that a HIP graph can capture.
// A launch covers a contiguous range of the table's fields and has one
// workgroup per work item (a column tile, or four strips of the horizontal
// adjoint at one level), which finds its field in the prefix sums and runs
// the same body as the single-field kernel.  The hardware dispatcher keeps
// the CUs filled: an earlier form whose resident workgroups pulled items
// from an atomic queue exposed each item's start (queue, search, argument
// block, first loads: several microseconds) on CUs that hold one or two
// workgroups, and ran every field in the largest class's registers.
#include <string.h>

#include "common.hpp"
#include "k_colsplit.hpp"
#include "k_hadj_strip.hpp"
#include "k_split.hpp"
#include "launch.hpp"

namespace gt4mi {

// ------------------------------------------------------------------ table upload
#ifdef GT4MI_UPLOAD
struct ByteChunk {
  uint32_t nwords;
  uint32_t words[960];
};

__global__ void __launch_bounds__(kWG) k_write_words(uint32_t* dst, ByteChunk c) {
  for (uint32_t t = threadIdx.x; t < c.nwords; t += kWG) dst[t] = c.words[t];
}

hipError_t launch_upload(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const uint32_t* w = static_cast<const uint32_t*>(src);
  const size_t nwords = (bytes + 3) / 4;
  for (size_t off = 0; off < nwords; off += 960) {
    ByteChunk c;
    c.nwords = (uint32_t)((nwords - off) < 960 ? (nwords - off) : 960);
    memcpy(c.words, w + off, c.nwords * 4);
    hipLaunchKernelGGL(k_write_words, dim3(1), dim3(kWG), 0, s, static_cast<uint32_t*>(dst) + off, c);
  }
  return hipGetLastError();
}
#endif

// ------------------------------------------------------------------ lookup
// The work list is written by the upload kernels before the launch and is
// the same for every lane: values read from it are taken from lane 0, so
// the field, its argument block and the buffer descriptors built from it
// are known to be uniform and stay in SGPRs.
__device__ __forceinline__ int uniform_ld(const int32_t* p) { return __builtin_amdgcn_readfirstlane(*p); }

template <typename S>
__device__ __forceinline__ S uniform_ld(const S* p) {
  static_assert(sizeof(S) % 4 == 0, "argument blocks are whole words");
  struct Words {
    uint32_t w[sizeof(S) / 4];
  } v;
  const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(S) / 4); ++i) v.w[i] = __builtin_amdgcn_readfirstlane(q[i]);
  return __builtin_bit_cast(S, v);
}

// Field of work item w among the n fields whose first items are at p: the
// last e with p[e] <= w.  The wave reads 64 prefixes at a time (one memory
// latency for up to 64 fields, where a binary search waits for five loads in
// a row) and counts those at or below w.
__device__ __forceinline__ int find_entry(const int32_t* __restrict__ p, int n, int w) {
  const int lane = threadIdx.x & 63;
  int at_or_below = 0;
  for (int b = 0; b < n; b += 64) {
    const int first = b + lane < n ? p[b + lane] : INT32_MAX;
    at_or_below += __popcll(__ballot(first <= w));
  }
  return at_or_below - 1;
}

// Work item of workgroup b of a launch of n: each XCD takes runs of 16 consecutive
// items, so that tiles that share halo rows share an L2; what does not fill a round of
// runs keeps the dispatch order.  Short runs, because a contiguous eighth of the items
// (xcd_tile) would leave the longest columns to one XCD.  Dispatch order against runs
// of 8, 16, 32, 64, us: FP32 10 fields 384x384x(96, 97) 706, 544, 536, 532, 534,
// 6 fields 300x300x130 371, 309, 307, 306, 311, 16 fields of 60-140 columns a side 92,
// 82, 82, 86, 87; FP64 6 fields 300x300x130 723 in dispatch order, 625 in runs of 16,
// 631 in runs of 64.
constexpr int kItemRun = 16;
__device__ __forceinline__ int run_item(int b, int n) {
  constexpr int round = kNumXcd * kItemRun;
  const int first = b / round * round;
  if (first + round > n) return b;
  return first + b % kNumXcd * kItemRun + b % round / kNumXcd;
}

// ------------------------------------------------------------------ kernels
// The fields of one launch may run different tile shapes (each field takes
// the tile that wastes the fewest lanes on its ragged edges): the work item
// runs the body of its field's tile, a uniform branch, in LDS shared by the
// three shapes.
template <typename T, int NT>
union BatchSmem {
  SplitSmem<T, 64, NT / 64> t64;
  SplitSmem<T, 32, NT / 32> t32;
  SplitSmem<T, 16, NT / 16> t16;
};

// Forward step, half-column register class NKH, tiles of NT columns.
template <typename T, int NT, int NKH, int PD, bool MASK>
__global__ void __launch_bounds__(2 * NT) k_step_batched(BatchRange r, const StepArgs<T>* __restrict__ ent) {
  __shared__ BatchSmem<T, NT> sm;
  const int w = r.first + run_item(blockIdx.x, gridDim.x);
  const int e = find_entry(r.prefix, r.n, w);
  const StepArgs<T> A = uniform_ld(ent + e);
  const int tile = w - uniform_ld(r.prefix + e);
  if (A.tile_i == 64)
    step_split_tile<T, 64, NT / 64, NKH, PD, MASK, 1>(A, tile, sm.t64);
  else if (A.tile_i == 32)
    step_split_tile<T, 32, NT / 32, NKH, PD, MASK, 1>(A, tile, sm.t32);
  else
    step_split_tile<T, 16, NT / 16, NKH, PD, MASK, 1>(A, tile, sm.t16);
}

// Column adjoint lambda = T^{-T} x_bar (argument blocks in column form).
template <typename T, int NKH>
__global__ void __launch_bounds__((2 * ColClass<T, NKH>::nt), (ColClass<T, NKH>::waves))
    k_vadj_batched(BatchRange r, const StepArgs<T>* __restrict__ ent) {
  constexpr int NT = ColClass<T, NKH>::nt, LST = ColClass<T, NKH>::lst;
  __shared__ ColSmem<T, NT, LST> sm;
  const int w = r.first + (int)blockIdx.x;
  const int e = find_entry(r.prefix, r.n, w);
  const StepArgs<T> A = uniform_ld(ent + e);
  column_split_tile<T, NKH, GT4MI_COL_PD, true, NT, LST>(A, w - uniform_ld(r.prefix + e), sm);
}

// Horizontal adjoint: one workgroup per work item (field, group of
// kStripsPerWG strips, level), as the single-field gather's grid; each wave
// walks its strip of the group (FP32 strips hold two columns per lane).
// Items cost the same, so each XCD takes one contiguous run of them and
// strips that share rows share an L2.
template <typename T>
__global__ void __launch_bounds__(kWG) k_hadj_batched(BatchRange r, const AdjArgs<T>* __restrict__ ent) {
  const int w = r.first + xcd_tile(blockIdx.x, gridDim.x);
  const int e = find_entry(r.prefix, r.n, w);
  const AdjArgs<T> A = uniform_ld(ent + e);
  const int local = w - uniform_ld(r.prefix + e);
  const int groups = (A.ntiles + kStripsPerWG - 1) / kStripsPerWG;
  const int g = local % groups, k = local / groups;
  const int t = __builtin_amdgcn_readfirstlane(g * kStripsPerWG + (int)(threadIdx.x >> 6));
  if (t < A.ntiles) {
    constexpr int TJ = strip_rows<T>(), PD = strip_pd<T>();
    if constexpr (sizeof(T) == 4) {
      // two columns per lane (uniform branches on the item's ni)
      if (A.ni > 1 && A.ni % 2 == 0) return hdiff_adjoint_strip2<TJ, PD, false, false, true>(A, t, k);
      if (A.ni > 1) return hdiff_adjoint_strip2<TJ, PD, false, true, true>(A, t, k);
    }
    hdiff_adjoint_strip<T, TJ, PD, false>(A, t, k);
  }
}

// ------------------------------------------------------------------ launchers
// One workgroup of `lanes` per work item.  A grid counts its lanes in 32 bits and a
// larger one is cut off without an error, so longer ranges take several launches
// (kernels number their items from r.first).
template <typename K, typename A>
static hipError_t launch_range(K kernel, int lanes, BatchRange r, const A* ent, hipStream_t s) {
  const int most = (int)(UINT32_MAX / (uint32_t)lanes);
  for (int left = r.items; left > 0; left -= most, r.first += most) {
    hipLaunchKernelGGL(kernel, dim3(left < most ? left : most), dim3(lanes), 0, s, r, ent);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
hipError_t launch_step_batched(int cls, const BatchRange& r, const StepArgs<T>* ent, bool mask, hipStream_t s) {
  auto go = [&](auto kernel, int nt) { return launch_range(kernel, 2 * nt, r, ent, s); };
#define GT4MI_BATCH_STEP(C)                                                                               \
  if (cls == C) {                                                                                         \
    using K = StepBatchClass<T, C>;                                                                       \
    return mask ? go(k_step_batched<T, K::nt, K::nkh, K::pd, true>, K::nt)                                \
                : go(k_step_batched<T, K::nt, K::nkh, K::pd, false>, K::nt);                              \
  }
  GT4MI_BATCH_STEP(0)
  GT4MI_BATCH_STEP(1)
  GT4MI_BATCH_STEP(2)
#undef GT4MI_BATCH_STEP
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_vadj_batched(int cls, const BatchRange& r, const StepArgs<T>* ent, hipStream_t s) {
  auto go = [&](auto kernel, int nt) { return launch_range(kernel, 2 * nt, r, ent, s); };
  // the host puts short FP32 columns into class 0, so it may stash no levels
  static_assert(sizeof(T) == 8 || ColClass<T, 72>::lst == 0);
  return cls == 0 ? go(k_vadj_batched<T, 72>, ColClass<T, 72>::nt) : go(k_vadj_batched<T, 48>, ColClass<T, 48>::nt);
}

template <typename T>
hipError_t launch_hadj_batched(const BatchRange& r, const AdjArgs<T>* ent, hipStream_t s) {
  return launch_range(k_hadj_batched<T>, kWG, r, ent, s);
}

#ifdef GT4MI_UPLOAD
int vadj_batched_tile_rows(bool f64, int cls) {
  if (f64) return (cls == 0 ? ColClass<double, 72>::nt : ColClass<double, 48>::nt) / 64;
  return (cls == 0 ? ColClass<float, 72>::nt : ColClass<float, 48>::nt) / 64;
}
#endif

// one object per element type (-DGT4MI_T=float|double); the float one also
// holds the table upload (-DGT4MI_UPLOAD)
template hipError_t launch_step_batched<GT4MI_T>(int, const BatchRange&, const StepArgs<GT4MI_T>*, bool, hipStream_t);
template hipError_t launch_vadj_batched<GT4MI_T>(int, const BatchRange&, const StepArgs<GT4MI_T>*, hipStream_t);
template hipError_t launch_hadj_batched<GT4MI_T>(const BatchRange&, const AdjArgs<GT4MI_T>*, hipStream_t);

}  // namespace gt4mi
