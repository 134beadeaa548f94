// k_param.hip -- gradients of one step with respect to its parameters
// (coeff and the vertical velocity w), for parameter tuning.
//
// With the limiter decisions held fixed the diffusion is h = u - coeff D(u),
// D the divergence of the limited fluxes (independent of coeff), and the
// column solve is T(w) x = h + data.  Given lam = T^{-T} x_bar (the step
// adjoint's data_bar) and the step's output x:
//   coeff_bar = -sum_p lam(p) D(u)(p)
//   w_bar_j   = r/4 [lam_j x_{j-1} - lam_{j-1} x_j - s_j (lam_j x_j + lam_{j-1} x_{j-1})]
// for the staggered levels j = 1 .. nk-1 (s_j = sign w_j, 0 at 0), the
// chain rule of dL/dT(k,l) = -lam_k x_l through a_j = -r/4 w_j,
// c_{j-1} = r/4 w_j and the |a|, |c| terms of the diagonal; w_0 and w_nk do
// not enter T and get 0.
#include <algorithm>

#include "k_hdiff_strip.hpp"
#include "k_step.hpp"
#include "launch.hpp"

namespace gt4mi {

// The workgroup's sum of its lanes' sums, to *out.
__device__ __forceinline__ void workgroup_sum(Sum2 s, Sum2* red, double* out) {
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) s.add(__shfl_down(s.hi, h), __shfl_down(s.lo, h));
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < kWG / 64; ++w) s.add(red[w].hi, red[w].lo);
  *out = s.value();
}

// Sum of lam * D(u) over the strips of one workgroup (k_hdiff_strip.hpp's walk)
// and a run of levels, in FP64, to partial[block] (fixed order: the result does
// not depend on scheduling).  A.data holds lam.  Bound by memory; with the final
// sum, against the tile form below, us: FP64 256x256x80 28.8, 38.2; 384x384x64 41.6,
// 48.1; 838x538x19 39.9, 47.2; FP32 21.1, 30.9; 26.2, 31.9; 23.8, 31.0.
template <typename T, int LANE>
__global__ void __launch_bounds__(kWG) k_coeff_partial(StepArgs<T> A, int levels, double* partial) {
  __shared__ Sum2 red[kStripsPerWG];
  const int wave = threadIdx.x >> 6;
  const int t = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * kStripsPerWG + wave);
  const int k0 = blockIdx.y * levels, k1 = min(k0 + levels, A.nk);
  Sum2 s{0.0, 0.0};
  if (t < A.ntiles)
    for (int k = k0; k < k1; ++k) {
      const Sum2 l = hdiff_strip_of<T, kHCoeffBar, LANE>(A, t, k);
      s.add(l.hi, l.lo);
    }
  workgroup_sum(s, red, partial + blockIdx.y * gridDim.x + blockIdx.x);
}

// The same sum over a 64 x 4 tile marched through every level, u in LDS (one barrier
// per level, the next level's loads in flight), to partial[tile].  For few levels on
// as many tiles as the chip holds, where the walk is bound by its rows' latencies
// (512x512x20: FP64 22.1 us against 29.1, FP32 14.4 against 20.8; 1000x500x8 19.0,
// 22.9 and 14.0, 18.2), and where the workspace holds no more than a sum per tile
// (57x111x66 27.6, 44.8 and 23.3, 31.7).
template <typename T>
__global__ void __launch_bounds__(kWG) k_coeff_tile(StepArgs<T> A, double* partial) {
  constexpr int TI = 64, TJ = kWG / TI;
  using TA = TileAddr<T, TI, TJ>;
  constexpr int HI = TA::HI, NLD = TA::NLD;
  __shared__ T su[2][NLD * kWG];
  __shared__ Sum2 red[kWG / 64];
  TA t;
  t.init(blockIdx.x, A.tiles_i, A.ni, A.nj, A.u_sj);
  const LevelView vu = level_view(A.u, A.u_sj, A.u_sk, -2, -2, A.nj + 4);
  const LevelView vl = level_view(A.data, A.d_sj, A.d_sk, 0, 0, A.nj);
  const uint32_t loff = ((uint32_t)t.ic + (uint32_t)t.jc * (uint32_t)A.d_sj) * (uint32_t)sizeof(T);
  const T gs = form_sign<T>(A.form);
  LevelCursor cur_u{vu.base, vu.level_bytes, vu.window}, cur_l{vl.base, vl.level_bytes, vl.window};
  T nu[NLD], nl;
  auto issue = [&](int k) {  // level k, the last one again past it
    const auto r = cur_u.rsrc();
#pragma unroll
    for (int q = 0; q < NLD; ++q) nu[q] = buf_ld(r, t.hoff[q], T());
    nl = buf_ld(cur_l.rsrc(), loff, T());
    const bool go = k + 1 < A.nk;
    cur_u.advance(go);
    cur_l.advance(go);
  };
  issue(0);
  Sum2 s{0.0, 0.0};
  for (int k = 0; k < A.nk; ++k) {
    T* U = su[k & 1];
#pragma unroll
    for (int q = 0; q < NLD; ++q) U[threadIdx.x + q * kWG] = nu[q];
    const T lam = nl;
    issue(k + 1);
    __syncthreads();
    bool kxr, kxl, kyr, kyl;
    const T div = limited_divergence(load_diamond<T, HI>(U + (t.tj + 2) * HI + (t.ti + 2)), gs, kxr, kxl, kyr, kyl);
    s.add_product(t.active ? lam : T(0), t.active ? gs * div : T(0));
  }
  workgroup_sum(s, red, partial + blockIdx.x);
}

// coeff_bar = -(sum of the partials), summed in a fixed order by one workgroup.
constexpr int kFinalWG = 1024;
__global__ void __launch_bounds__(kFinalWG) k_coeff_final(const double* partial, int n, void* coeff_bar, bool f32) {
  __shared__ Sum2 red[kFinalWG / 64];
  const int tid = threadIdx.x;
  Sum2 s{0.0, 0.0};
  for (int p = tid; p < n; p += kFinalWG) s.add(partial[p], 0.0);
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) s.add(__shfl_down(s.hi, h), __shfl_down(s.lo, h));
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  if (tid) return;
  for (int w = 1; w < kFinalWG / 64; ++w) s.add(red[w].hi, red[w].lo);
  const double v = n > 0 ? -s.value() : 0.0;
  if (f32) *static_cast<float*>(coeff_bar) = (float)v;
  else *static_cast<double*>(coeff_bar) = v;
}

// w_bar of L staggered levels of a 64 x 4 tile's columns, a lane per column, every
// load in flight before the first use; the level below is read again by the run
// below.  Bound by memory (FP64 512x512x80 114 us: 5.9 TB/s of the four streams).
// One lane marching its column a level ahead kept too little in flight: FP64
// 512x512x80 124 us, 256x256x80 53 (31 here), 301x203x137 91 (51); FP32 70 (60), 44
// (14), 76 (28).  Runs of one tile side by side on an XCD were slower (130 us).
template <typename T, int L>
__global__ void __launch_bounds__(kWG) k_w_grad(WGradArgs<T> A) {
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int bi = tile % A.tiles_i, bj = tile / A.tiles_i;
  const int i = bi * 64 + (threadIdx.x & 63), j = bj * 4 + (threadIdx.x >> 6);
  const bool active = i < A.ni && j < A.nj;
  const int ic = min(i, A.ni - 1), jc = min(j, A.nj - 1);
  constexpr uint32_t S = sizeof(T);
  const LevelView vw = level_view(A.w, A.w_sj, A.w_sk, 0, 0, A.nj);
  const LevelView vx = level_view(A.x, A.x_sj, A.x_sk, 0, 0, A.nj);
  const LevelView vl = level_view(A.lam, A.l_sj, A.l_sk, 0, 0, A.nj);
  const LevelView vb = level_view<T>(A.wbar, A.b_sj, A.b_sk, 0, 0, A.nj);
  const uint32_t woff = ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.w_sj) * S;
  const uint32_t xoff = ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.x_sj) * S;
  const uint32_t loff = ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.l_sj) * S;
  const uint32_t boff = active ? ((uint32_t)ic + (uint32_t)jc * (uint32_t)A.b_sj) * S : kOffNone;
  const int nk = A.nk;
  if (nk < 1) {  // one staggered level, no column
    buf_st(vb.at(0), boff, T(0));
    return;
  }
  for (int k0 = blockIdx.y * L; k0 <= nk; k0 += gridDim.y * L) {
    T l[L + 1], x[L + 1], w[L];
#pragma unroll
    for (int n = 0; n <= L; ++n) {  // levels k0 - 1 .. k0 + L - 1 (clamped: an edge level's value goes unused)
      const int k = max(min(k0 + n - 1, nk - 1), 0);
      l[n] = buf_ld(vl.at(k), loff, T());
      x[n] = buf_ld(vx.at(k), xoff, T());
      if (n) w[n - 1] = buf_ld(vw.at(min(k0 + n - 1, nk)), woff, T());
    }
    pin_prefetch();
#pragma unroll
    for (int n = 0; n < L; ++n) {
      const int k = k0 + n;
      if (k > nk) break;  // uniform
      const T s = w[n] > T(0) ? T(1) : (w[n] < T(0) ? T(-1) : T(0));
      const T g = A.q * ((l[n + 1] * x[n] - l[n] * x[n + 1]) - s * (l[n + 1] * x[n + 1] + l[n] * x[n]));
      // w_0 and w_nk do not enter T
      buf_st(vb.at(k), boff, k == 0 || k == nk ? T(0) : g);
    }
  }
}

// ------------------------------------------------------------------ launchers
int64_t coeff_partial_most(bool f64, int64_t ni, int64_t nj, int64_t nk) {
  const int64_t w = f64 ? kHStripOut : kHStripOut2;
  constexpr int R = HStrip<kHCoeffBar, 1>::rows;
  const int64_t strips = ((ni + w - 1) / w) * ((nj + R - 1) / R);
  return (strips + kStripsPerWG - 1) / kStripsPerWG * std::min<int64_t>(nk, kMaxGridY);
}

// Whether the sum takes the tile form: estimated times, us, fitted to 60 sizes (of 8
// to 140 levels) in each type.  The tile form: a level costs what the tiles on a CU
// take, from one to four of them, and again for every 1024 tiles.  The walk: rounds
// of 256 workgroups and, where the workspace leaves `levels` of them to a workgroup,
// a chain of strips.  The faster form or one within 10% of it nearly everywhere
// (512x512x80 takes the walk: FP64 86 against 81, FP32 49 against 53).
static bool coeff_by_tiles(bool f64, int64_t tiles, int64_t wgs, int64_t nk, int64_t levels) {
  static const double level_us[2][5] = {{0, 0.29, 0.34, 0.41, 0.55}, {0, 0.33, 0.52, 0.66, 1.0}};
  const double* us = level_us[f64];
  const double tile = 6.0 + nk * (us[4] * (tiles / (4 * kCus)) + us[(tiles % (4 * kCus) + kCus - 1) / kCus]);
  double walk = 9.0 + 3.0 * ((wgs * nk + kCus - 1) / kCus);
  if (levels > 1) {
    const double chain = 8.0 + (f64 ? 4.1 : 4.6) * levels;
    walk = std::max(walk, chain) + 0.1 * std::min(walk, chain);
  }
  return std::max(tile, 12.0) < walk;
}

template <typename T>
hipError_t launch_param_grads(const StepArgs<T>& Ain, const WGradArgs<T>* W, double* partial, int64_t slots,
                              void* coeff_bar, bool f32, hipStream_t s) {
  StepArgs<T> A = Ain;
  const bool some = A.ni > 0 && A.nj > 0;
  if (coeff_bar) {
    int n = 0;
    if (some && A.nk > 0) {
      hdiff_strip_lanes(A, [&](auto lane) { hdiff_strip_count<T, kHCoeffBar, decltype(lane)::value>(A); });
      // a run per level, or as many runs as the partials have room for (at least
      // one: a strip workgroup covers more columns than a 64 x 4 tile)
      const int64_t wgs = (A.ntiles + kStripsPerWG - 1) / kStripsPerWG;
      const int runs = (int)std::min<int64_t>({A.nk, slots / wgs, kMaxGridY});
      const int levels = (A.nk + runs - 1) / runs;
      const int64_t tiles = coeff_partial_least(A.ni, A.nj);
      if (tiles <= UINT32_MAX / kWG && coeff_by_tiles(sizeof(T) == 8, tiles, wgs, A.nk, levels)) {
        A.tiles_i = (A.ni + 63) / 64;
        n = (int)tiles;
        hipLaunchKernelGGL(k_coeff_tile<T>, dim3(n), dim3(kWG), 0, s, A, partial);
      } else {
        const dim3 grid((uint32_t)wgs, (A.nk + levels - 1) / levels);
        n = (int)(grid.x * grid.y);
        hdiff_strip_lanes(A, [&](auto lane) {
          hipLaunchKernelGGL((k_coeff_partial<T, decltype(lane)::value>), grid, dim3(kWG), 0, s, A, levels, partial);
        });
      }
    }
    hipLaunchKernelGGL(k_coeff_final, dim3(1), dim3(kFinalWG), 0, s, partial, n, coeff_bar, f32);
  }
  if (W && some) {
    WGradArgs<T> B = *W;
    B.tiles_i = (B.ni + 63) / 64;
    const int nt = B.tiles_i * ((B.nj + 3) / 4);
    auto go = [&](auto levels) {
      constexpr int L = decltype(levels)::value;
      const int runs = B.nk / L + 1;  // of the nk + 1 staggered levels
      hipLaunchKernelGGL((k_w_grad<T, L>), dim3(nt, std::min(runs, kMaxGridY)), dim3(kWG), 0, s, B);
    };
    // Levels per run: each run reads one level of lam and x again, but more of them
    // keep more streams of HBM open.  2, 3, 4, 8, us: FP64 512x512x80 118, 124, 128,
    // 136; fields that stay in the cache 219x604x36 27.3, 25.7, 25.1, 23.9 (one lane a
    // column 22.8), 435x231x65 37.6, 34.3, 33.5, 32.3.  A last run of one level costs a
    // whole one (FP32 1000x500x8 14.1, 11.6, 13.2, 15.0; one lane a column 11.3): of
    // three and four, what takes fewer accesses.
    const bool large = sizeof(T) == 8 && 4 * (int64_t)B.ni * B.nj * B.nk * 8 > (int64_t)320 << 20;
    auto accesses = [&](int L) { return (int64_t)(B.nk / L + 1) * (4 * L + 2); };
    if (large) go(std::integral_constant<int, 2>{});
    else if (accesses(3) < accesses(4)) go(std::integral_constant<int, 3>{});
    else go(std::integral_constant<int, 4>{});
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_coeff_field_grad(const StepArgs<T>& A, hipStream_t s) {
  if (A.ni <= 0 || A.nj <= 0 || A.nk <= 0) return hipGetLastError();
  for (int k = 0; k < A.nk; k += kMaxGridY) {  // one grid row per level
    StepArgs<T> B = A;
    B.u += (int64_t)k * A.u_sk;
    B.data += (int64_t)k * A.d_sk;
    B.out += (int64_t)k * A.o_sk;
    B.nk = std::min(A.nk - k, kMaxGridY);
    const hipError_t e = launch_hdiff_strip<T, kHKappaBar>(B, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template hipError_t launch_coeff_field_grad<float>(const StepArgs<float>&, hipStream_t);
template hipError_t launch_coeff_field_grad<double>(const StepArgs<double>&, hipStream_t);
template hipError_t launch_param_grads<float>(const StepArgs<float>&, const WGradArgs<float>*, double*, int64_t, void*, bool,
                                              hipStream_t);
template hipError_t launch_param_grads<double>(const StepArgs<double>&, const WGradArgs<double>*, double*, int64_t, void*, bool,
                                               hipStream_t);

}  // namespace gt4mi
