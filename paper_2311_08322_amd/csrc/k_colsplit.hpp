// k_colsplit.hpp -- the column solves alone (vertical advection and its
// adjoint), each column eliminated from both ends by two lanes.
//
// Forward:  T x = u + data.  Adjoint:  T^T lambda = x_bar.
// T^T is tridiagonal with sub-diagonal c_{k-1}, diagonal b_k and
// super-diagonal a_{k+1}; in terms of w the near/far coefficients of the two
// sweeps (see k_split.hpp) are those of T with the sign flipped:
//   top, level k:    near = c_{k-1} = +r/4 w_k,      far = a_{k+1} = -r/4 w_{k+1}
//   bottom, level k: near = a_{k+1} = -r/4 w_{k+1},  far = c_{k-1} = +r/4 w_k
// while the diagonal b_k = 1 + |a_k| + |c_k| = 1 + |near| + |far| is the same.
// So both solves are one kernel: a sign and the right-hand side differ.
//
// Bound by HBM (three or four streams, each touched once).  e and f of every
// level stay on the CU until the back substitution: e in VGPRs, f in VGPRs
// except for the LST outermost levels of each half, whose f sits in LDS (one
// 8- or 4-byte word per lane and level, no bank conflicts).  The outermost
// levels are eliminated first and substituted last, so their LDS words are
// read in one straight run at the end.  LDS is otherwise idle here, and what
// it takes off the VGPRs decides how many waves a SIMD holds.
#pragma once

#include "k_step.hpp"

#include <type_traits>

// Levels loaded ahead by the column-only kernels (two loads per level, so
// they can run further ahead than the fused step at the same registers).
#ifndef GT4MI_COL_PD
#define GT4MI_COL_PD 2
#endif

namespace gt4mi {

// NT: columns of the workgroup's tile (64 wide, NT/64 rows), two lanes each.
template <typename T, int NT, int LST>
struct ColSmem {
  T xch[2][2][NT];                  // innermost (e, f) of each half and column
  T st[LST > 0 ? LST : 1][2 * NT];  // f of the outermost levels (LST > 0)
};

// Every half eliminates at least LST levels (A.nk / 2 >= LST: the host's
// register classes see to it), so the stashed levels need no check.
template <typename T, int NKH, int PD, bool ADJ, int NT, int LST>
__device__ __forceinline__ void column_split_tile(const StepArgs<T>& A, int tile, ColSmem<T, NT, LST>& sm) {
  constexpr int TJ = NT / 64;
  const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);  // 0: top, 1: bottom
  const int ltid = threadIdx.x - half * NT;
  const int bi = tile % A.tiles_i, bj = tile / A.tiles_i;
  const int i = bi * 64 + (ltid & 63), j = bj * TJ + (ltid >> 6);
  const bool active = (i < A.ni) && (j < A.nj);
  const int ic = min(i, A.ni - 1), jc = min(j, A.nj - 1);
  const int nk = A.nk, m = nk / 2;
  const int nlev = half ? nk - m : m;
  const int nsteps = nk - m;
  const int k0 = half ? nk - 1 : 0, dir = half ? -1 : 1;
  constexpr uint32_t S = sizeof(T);
  // forward: u (rhs part 1), data (part 2); adjoint: u holds x_bar, data unused
  const LevelView vu = level_view(A.u, A.u_sj, A.u_sk, 0, 0, A.nj);
  const LevelView vd = level_view(A.data, A.d_sj, A.d_sk, 0, 0, A.nj);
  const LevelView vw = level_view(A.w, A.w_sj, A.w_sk, 0, 0, A.nj);
  const LevelView vo = level_view<T>(A.out, A.o_sj, A.o_sk, 0, 0, A.nj);
  const uint32_t uoff = ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.u_sj) * S;
  const uint32_t doff = ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.d_sj) * S;
  const uint32_t woff = ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.w_sj) * S;
  const uint32_t ooff = active ? ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.o_sj) * S : kOffNone;

  LevelCursor cur_u{vu.base + (int64_t)k0 * vu.level_bytes, dir * vu.level_bytes, vu.window};
  LevelCursor cur_d{vd.base + (int64_t)k0 * vd.level_bytes, dir * vd.level_bytes, vd.window};
  LevelCursor cur_w{vw.base + (int64_t)(half ? k0 : 1) * vw.level_bytes, dir * vw.level_bytes, vw.window};
  T pr[PD], pw[PD];
  auto issue = [&](int slot, int s) {
    T r = buf_ld(cur_u.rsrc(), uoff, T());
    if constexpr (!ADJ) r += buf_ld(cur_d.rsrc(), doff, T());
    pr[slot] = r;
    pw[slot] = buf_ld(cur_w.rsrc(), woff, T());
    const bool go = s + 1 < nlev;
    cur_u.advance(go);
    if constexpr (!ADJ) cur_d.advance(go);
    cur_w.advance(go);
  };
#pragma unroll
  for (int s = 0; s < PD; ++s) issue(s, s);

  T ev[NKH];
  T fv[NKH];
  T wp = T(0), e = T(0), f = T(0);
  const T sn = (half ? A.r4 : -A.r4) * (ADJ ? T(-1) : T(1));
#pragma unroll
  for (int s = 0; s < NKH; ++s) {
    if (s >= nsteps) break;  // uniform; the only branch, so load counters stay exact
    __builtin_amdgcn_sched_barrier(0);
    const int slot = s % PD;
    const T rhs = pr[slot], wn = pw[slot];
    if (s + PD < NKH) issue(slot, s + PD);
    pin_prefetch();
    const bool act = s < nlev;
    const int k = k0 + dir * s;
    const T nr = (s > 0) ? sn * wp : T(0);
    const T fr = (half == 0 || k > 0) ? -sn * wn : T(0);
    const T b = T(1) + absv(nr) + absv(fr);
    const T inv = recip(b - nr * e);
    const T en = fr * inv;
    const T fn = (rhs - nr * f) * inv;
    e = act ? en : e;
    f = act ? fn : f;
    wp = act ? wn : wp;
    ev[s] = e;
    if (s < LST) sm.st[s][threadIdx.x] = f;  // read back by the same lane
    else fv[s] = f;
  }
  sm.xch[half][0][ltid] = e;
  sm.xch[half][1][ltid] = f;
  __syncthreads();
  const T eo = sm.xch[1 - half][0][ltid], fo = sm.xch[1 - half][1][ltid];
  const T et = half ? eo : e, ft = half ? fo : f;
  const T eb = half ? e : eo, fb = half ? f : fo;
  const T xm = (fb - eb * ft) * recip(T(1) - eb * et);
  const T xm1 = ft - et * xm;
  T x = half ? xm1 : xm;
#pragma unroll
  for (int s = NKH - 1; s >= LST; --s) {
    if (s < nlev) {
      const auto ro = vo.at(k0 + dir * s);
      x = fv[s] - ev[s] * x;
      buf_st(ro, ooff, x);
    }
  }
#pragma unroll
  for (int s = LST - 1; s >= 0; --s) {
    const auto ro = vo.at(k0 + dir * s);
    x = sm.st[s][threadIdx.x] - ev[s] * x;
    buf_st(ro, ooff, x);
  }
}

// The register classes: half-columns of up to `nkh` levels in tiles of NT
// columns with LST levels' f in LDS.  A class's columns have more than twice
// the previous class's levels, so every half holds more than that many and
// LST may not exceed it.  Measured on cold buffers, 512x512 columns:
//   FP64, 97..144 levels: f of 36 levels in LDS lets e and f of the whole
//     column stay on chip at two waves per SIMD (2 x 80 KB of LDS per CU);
//     with f staged in the output instead (read back in the substitution)
//     the adjoint at 137 levels took 242 us against 190, the forward solve
//     306 against 237.
//   FP64, up to 96 levels: three waves per SIMD (10 to 25 levels in LDS) were
//     no faster than two (109.8 against 108.6 us at 80): memory bound.
//   FP32, 49..80 levels: 20 levels in LDS make room for six waves per SIMD
//     (56.2 against 58.9 us with four).
//   FP32, 97..144: 128-column tiles hold three workgroups per CU (three waves
//     per SIMD) where 256-column tiles of 160 levels held two waves: 97.8
//     against 104.5 us at 137.
template <typename T, int NKH>
struct ColClass {
  static constexpr int nt = 256, lst = 0, waves = 2;
};
template <>
struct ColClass<double, 72> {
  static constexpr int nt = 128, lst = 36, waves = 2;
};
template <>
struct ColClass<float, 40> {
  static constexpr int nt = 128, lst = 20, waves = 6;
};
template <>
struct ColClass<float, 48> {
  static constexpr int nt = 256, lst = 0, waves = 4;
};
template <>
struct ColClass<float, 72> {
  static constexpr int nt = 128, lst = 0, waves = 3;
};

template <typename T, int NKH, int PD, bool ADJ>
__global__ void __launch_bounds__((2 * ColClass<T, NKH>::nt), (ColClass<T, NKH>::waves)) k_column_split(StepArgs<T> A) {
  constexpr int NT = ColClass<T, NKH>::nt, LST = ColClass<T, NKH>::lst;
  __shared__ ColSmem<T, NT, LST> sm;
  column_split_tile<T, NKH, PD, ADJ, NT, LST>(A, xcd_tile(blockIdx.x, gridDim.x), sm);
}

// longest column of the two-ended solves: FP64 144 levels, FP32 160
template <typename T, bool ADJ>
hipError_t launch_column_split_classes(StepArgs<T> A, hipStream_t s) {
  A.tiles_i = (A.ni + 63) / 64;
  const int nkh = A.nk - A.nk / 2;
  auto go = [&](auto cls) {
    constexpr int N = decltype(cls)::value, NT = ColClass<T, N>::nt, TJ = NT / 64;
    A.ntiles = A.tiles_i * ((A.nj + TJ - 1) / TJ);
    hipLaunchKernelGGL((k_column_split<T, N, GT4MI_COL_PD, ADJ>), dim3(A.ntiles), dim3(2 * NT), 0, s, A);
    return hipGetLastError();
  };
  if (nkh <= 16) return go(std::integral_constant<int, 16>{});
  if (nkh <= 24) return go(std::integral_constant<int, 24>{});
  if constexpr (sizeof(T) == 4)
    if (nkh <= 40) return go(std::integral_constant<int, 40>{});
  if (nkh <= 48) return go(std::integral_constant<int, 48>{});
  if (nkh <= 72) return go(std::integral_constant<int, 72>{});
  if constexpr (sizeof(T) == 4)
    if (nkh <= 80) return go(std::integral_constant<int, 80>{});
  return hipErrorInvalidValue;
}

}  // namespace gt4mi
