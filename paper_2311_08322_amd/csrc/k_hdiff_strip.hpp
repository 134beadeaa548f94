// k_hdiff_strip.hpp -- the horizontal diffusion alone and the coefficient's
// gradients, as a row walk.
//
// Per level, on the interior:
//   lap(p)  = 4 u(p) - ((u(p - e_i) + u(p + e_i)) + (u(p - e_j) + u(p + e_j)))
//   fx(q)   = lap(q + e_i) - lap(q), kept unless fx * (u(q + e_i) - u(q)) > 0
//   fy(q)   = lap(q + e_j) - lap(q), kept likewise with u(q + e_j) - u(q)
//   out(p)  = u(p) - coeff ((Fx(p) - Fx(p - e_i)) + (Fy(p) - Fy(p - e_j)))
// with the same association as the tile kernel, so values and limiter bits
// are the same bit for bit.
//
// One wavefront owns 64 consecutive i (lane = i) of one level and walks
// 8 + 4 rows in j (HStrip), one u row loaded per step PD rows ahead; neighbours in i
// come from DPP wave shifts, neighbours in j from the rows already walked.
// Per step it forms lap of the row before the newest, its x fluxes, the y
// fluxes below it, and out of the row two back: every value once.  Lanes
// 4..59 own the strip's 56 output columns, which start on a byte of the
// mask rows, so a strip writes its limiter bits as whole bytes (a wave
// ballot) and strips never share a byte.  No LDS, no barriers.
//
// The same walk, with a second interior field read row by row beside u:
//   kHVar       the generalised diffusion (per-point coefficient kappa or the
//               scalar; the form's sign on limiter and coefficient)
//   kHKappaBar  out(p) = -lam(p) D(u)(p), D the divergence of the kept fluxes
//   kHCoeffBar  the sum of lam(p) D(u)(p) over the strip
// (the form's sign folded in as in hdiff_var_of).  Bound by memory, like the
// plain walk.  Times on cold buffers against tile kernels that staged u in LDS
// behind a barrier per level, 512x512x80 and 256x256x80: FP64 kappa field 111 ->
// 98 and 28.6 -> 29.6 us, damping 94 -> 75 and 25.7 -> 23.4, kappa_bar 105 -> 95.5
// (5.3 TB/s) and 49 -> 29; FP32 59 -> 53 and 16.4 -> 16.0, 53 -> 40 and 13.8 ->
// 13.3, 59 -> 53 and 36 -> 16.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace gt4mi {

constexpr int kHStripOut = 56;   // output columns per strip: 7 bytes of a mask row
// Output rows of a strip and rows in flight ahead of their use, by what the walk
// does and its columns per lane (LANE below).  Eight rows with all twelve input
// rows in flight against 16 and 4 (5 with a second field), on cold buffers: FP64
// 512x512x80 67 against 68.5 us, with the mask 74 / 76, kappa field 92.5 / 96;
// 256x256x80 19.0 / 20.4, 22.4 / 24.4, 27.5 / 29.3; FP32 with odd rows 501x403x60
// 23.5 / 26.2 and 29 / 34.3, kappa field 512x512x80 50.7 / 53.2.  FP32 in aligned
// pairs keeps 16 and 4 (256x256x80 10.7 against 11.3, with the mask 15.9 / 16.4),
// as does the sum, which only reads (FP64 512x512x80 95 against 117 us, 3.9 TB/s:
// what plain read streams reach).
enum HdiffMode { kHPlain, kHVar, kHKappaBar, kHCoeffBar };
template <int MODE, int LANE>
struct HStrip {
  static constexpr bool few = MODE == kHCoeffBar || (MODE == kHPlain && LANE == 2);
  static constexpr int rows = few ? 16 : 8, pd = few ? 4 : 12;
};

// A sum carried to twice the precision of binary64: hi is the plain sum, lo what
// its additions rounded off (Knuth's TwoSum), so that the order of the addends,
// which the domain's split fixes, does not show in the result.  Where hi is not
// finite, lo means nothing.
struct Sum2 {
  double hi, lo;
  __device__ __forceinline__ void add(double p, double e) {
#pragma clang fp contract(off)
    const double t = hi + p, z = t - hi;
    lo += ((hi - (t - z)) + (p - z)) + e;
    hi = t;
  }
  __device__ __forceinline__ void add_product(double a, double b) {
#pragma clang fp contract(off)
    const double p = a * b;
    add(p, __builtin_fma(a, b, -p));
  }
  // binary32 factors: the product is exact, and the plain sum's error (1e-16 of
  // it) is far below the factors' own rounding
  __device__ __forceinline__ void add_product(float a, float b) { hi += (double)a * (double)b; }
  __device__ __forceinline__ double value() const { return __builtin_isfinite(hi) ? hi + lo : hi; }
};

// the second field of a mode: kappa (VAR) or lam, which sits in the data slot
template <int MODE, typename T>
struct HdiffSecond {
  const char* base = nullptr;
  int64_t row = 0, level = 0;  // bytes
  bool has = false;
  __device__ __forceinline__ explicit HdiffSecond(const StepArgs<T>& A) {
    if constexpr (MODE == kHVar) {
      has = A.kappa != nullptr;
      base = reinterpret_cast<const char*>(A.kappa);
      row = A.c_sj * (int64_t)sizeof(T);
      level = A.c_sk * (int64_t)sizeof(T);
    } else if constexpr (MODE != kHPlain) {
      has = true;
      base = reinterpret_cast<const char*>(A.data);
      row = A.d_sj * (int64_t)sizeof(T);
      level = A.d_sk * (int64_t)sizeof(T);
    }
  }
};

// The strip `t` (A.tiles_i strips in i times the row blocks in j) at level k.
// Returns the lane's share of the sum (kHCoeffBar).
template <typename T, int TJ, int PD, int MODE>
__device__ __forceinline__ Sum2 hdiff_strip(const StepArgs<T>& A, int t, int k) {
  static_assert((TJ + 4) % PD == 0, "the row walk is unrolled by the prefetch depth");
  constexpr uint32_t S = sizeof(T);
  const int lane = threadIdx.x & 63;
  const int si = t % A.tiles_i, sj = t / A.tiles_i;
  const int ni = A.ni, nj = A.nj;
  const int i = kHStripOut * si - 4 + lane;  // lane 4 is the strip's first output column
  const int j0 = TJ * sj;                    // first output row
  const bool own = lane >= 4 && lane < 4 + kHStripOut && i < ni;
  constexpr bool SUM = MODE == kHCoeffBar;
  const bool has_mask = (MODE == kHPlain || MODE == kHVar) && A.mask != nullptr;
  const T coeff = MODE == kHPlain || MODE == kHVar ? step_coeff(A) : T(0);
  const T gs = MODE == kHPlain ? T(1) : form_sign<T>(A.form);
  const HdiffSecond<MODE, T> second(A);
  Sum2 sum{0.0, 0.0};

  // One descriptor per row (uniform base, a window of the row's width, empty
  // for a row outside the field) and a lane offset fixed for the walk.
  const auto row_rsrc = [&](const char* base, int64_t row_bytes, int r, int rows, uint32_t width) {
    const bool in = r >= 0 && r < rows;
    return make_rsrc(base + (in ? (int64_t)r * row_bytes : 0), in ? width : 0u);
  };
  const char* ubase = reinterpret_cast<const char*>(A.u) + ((int64_t)k * A.u_sk - 2 - 2 * A.u_sj) * S;
  const char* obase = reinterpret_cast<const char*>(A.out) + (int64_t)k * A.o_sk * S;
  const uint32_t u_off = (i >= -2 && i < ni + 2) ? (uint32_t)(i + 2) * S : kOffNone;  // window: ni + 4
  const uint32_t o_off = own ? (uint32_t)i * S : kOffNone;                            // window: ni
  // The limiter bits: one descriptor over the whole mask (the host sends
  // masks below 4 GiB here), so one byte store writes a row's x bytes
  // (lanes 0..6) and y bytes (lanes 8..14) together.
  const auto rm = make_rsrc(A.mask, has_mask ? (uint32_t)A.ml.total : 0u);
  const int64_t W = A.ml.words, plane_xy = (int64_t)nj * W * 8;
  const int64_t x_lev = A.ml.x_off + (int64_t)k * plane_xy, y_lev = A.ml.y_off + (int64_t)k * plane_xy;
  const int mb = lane & 7;                                  // the lane's byte of the strip's 7
  const bool xlane = lane < 7, ylane = lane >= 8 && lane < 15;
  const uint32_t mcol = (uint32_t)(kHStripOut / 8 * si + mb);  // byte within a mask row
  const bool mcol_in = mcol < (uint32_t)(W * 8);
  const int byte_shift = 4 + 8 * mb;
  const uint32_t ex_base = (uint32_t)(A.ml.ex_off + (int64_t)k * nj), ey_base = (uint32_t)(A.ml.ey_off + (int64_t)k * ni);

  T pu[PD];
  [[maybe_unused]] T p2[MODE == kHPlain ? 1 : PD];
  const int r0 = j0 - 2;
  constexpr int NR = TJ + 4;
  // u of row r, and the second field of row r - 2, which the step that takes
  // row r's slot completes
  auto issue = [&](int r, int s) {
    pu[s] = buf_ld(row_rsrc(ubase, A.u_sj * S, r + 2, nj + 4, (uint32_t)(ni + 4) * S), u_off, T());
    if constexpr (MODE != kHPlain)
      p2[s] = buf_ld(row_rsrc(second.base + k * second.level, second.row, r - 2, second.has ? nj : 0, (uint32_t)ni * S), o_off, T());
  };

  // the walk's state: u of rows R-1 and R-2, lap of row R-2, the kept x
  // fluxes of row R-2 and the kept y fluxes between rows R-3 and R-2
  T u1 = T(0), u2 = T(0), lap2 = T(0), Fx2 = T(0), Fy3 = T(0);
  auto step = [&](int n, int s, bool refill) {
    const int R = r0 + n;
    T uR = pu[s];
    asm volatile("" : "+v"(uR));  // a copy of its own: the slot is free for the refill
    [[maybe_unused]] T x2 = T(0);
    if constexpr (MODE != kHPlain) {
      x2 = p2[s];
      asm volatile("" : "+v"(x2));
    }
    if (refill) issue(R + PD, s);
    // the shifts run with every lane active (a disabled lane would read as 0)
    const T ue1 = lane_shift<kDppWaveShl1>(u1), uw1 = lane_shift<kDppWaveShr1>(u1);
    const T lap1 = T(4) * u1 - ((uw1 + ue1) + (u2 + uR));  // lap(R-1)
    const T lape1 = lane_shift<kDppWaveShl1>(lap1);
    const T Fxw2 = lane_shift<kDppWaveShr1>(Fx2);
    const T fx = lape1 - lap1;  // x flux of row R-1
    const bool kx = flux_kept(fx, gs * (ue1 - u1));
    const T Fx1 = kx ? fx : T(0);
    const T fy = lap1 - lap2;  // y flux between rows R-2 and R-1
    const bool ky = flux_kept(fy, gs * (u1 - u2));
    const T Fy2 = ky ? fy : T(0);
    const int q = R - 2;  // out(R-2)
    const T div = (Fx2 - Fxw2) + (Fy2 - Fy3);
    const bool qrow = q >= j0 && q < j0 + TJ;  // uniform
    if constexpr (SUM) {
      if (qrow && q < nj) sum.add_product(own ? x2 : T(0), own ? gs * div : T(0));
    }
    T v;
    if constexpr (MODE == kHPlain) v = u2 - coeff * div;
    else if constexpr (MODE == kHVar) v = u2 - (gs * (second.has ? x2 : coeff)) * div;
    else v = -(x2 * (gs * div));
    if (!SUM && qrow) buf_st(row_rsrc(obase, A.o_sj * S, q, nj, (uint32_t)ni * S), o_off, v);
    if (has_mask) {
      // x bits of row R-1 and y bits between rows R-2 and R-1, one store
      const int rx = R - 1;
      const uint64_t bx = __ballot(own && kx), by = __ballot(own && ky);
      const bool xrow = rx >= j0 && rx < j0 + TJ && rx < nj, yrow = qrow && q < nj;  // uniform
      uint32_t off = kOffNone;
      if (xlane && xrow && mcol_in) off = (uint32_t)(x_lev + (int64_t)rx * W * 8) + mcol;
      if (ylane && yrow && mcol_in) off = (uint32_t)(y_lev + (int64_t)q * W * 8) + mcol;
      buf_st_u8(rm, off, (uint8_t)((ylane ? by : bx) >> byte_shift));
      // the x flux at i = -1 and the y flux below row 0 have byte planes of their own
      if (si == 0 && xrow && rx >= 0) buf_st_u8(rm, i == -1 ? ex_base + (uint32_t)rx : kOffNone, kx ? 1 : 0);
      if (q == -1) buf_st_u8(rm, own ? ey_base + (uint32_t)i : kOffNone, ky ? 1 : 0);
    }
    Fy3 = Fy2;
    Fx2 = Fx1;
    lap2 = lap1;
    u2 = u1;
    u1 = uR;
  };

#pragma unroll
  for (int s = 0; s < PD; ++s) issue(r0 + s, s);
  int n = 0;
  for (; n < NR - PD; n += PD) {
#pragma unroll
    for (int s = 0; s < PD; ++s) step(n + s, s, true);
  }
#pragma unroll
  for (int s = 0; s < PD; ++s) step(n + s, s, false);
  if constexpr (MODE == kHPlain || MODE == kHVar) keep_coeff(A, coeff, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6));
  return sum;
}

// FP32: two adjacent columns per lane (a = 120 s - 4 + 2 l, b = a + 1), 128
// columns per wave of which lanes 2..61 own the strip's 120 output columns
// (15 bytes of a mask row).  The east neighbour of a and the west neighbour
// of b are in the lane itself, so a row needs half the shifts; the two
// columns' limiter bits come from two ballots, interleaved into the row's
// bytes.  Same values and bits as hdiff_strip.
constexpr int kHStripOut2 = 120;

// bits 0..3 of v to bits 0, 2, 4, 6
__device__ __forceinline__ uint32_t spread4(uint32_t v) {
  return (v & 1u) | ((v & 2u) << 1) | ((v & 4u) << 2) | ((v & 8u) << 3);
}

// ni >= 2; ODD: ni is odd, so the last lane's pair ends at the row's end
// (pair_at).  Reading odd rows column by column took 30.2 us at 501x403x60
// against 26.2.
template <int TJ, int PD, int MODE, bool ODD>
__device__ __forceinline__ Sum2 hdiff_strip2(const StepArgs<float>& A, int t, int k) {
  static_assert((TJ + 4) % PD == 0, "the row walk is unrolled by the prefetch depth");
  using T = float;
  constexpr uint32_t S = 4;
  const int lane = threadIdx.x & 63;
  const int si = t % A.tiles_i, sj = t / A.tiles_i;
  const int ni = A.ni, nj = A.nj;
  const int ia = kHStripOut2 * si - 4 + 2 * lane, ib = ia + 1;  // lane 2's a is the first output column
  const int j0 = TJ * sj;
  const bool owna = lane >= 2 && lane < 2 + kHStripOut2 / 2 && ia < ni;
  const bool ownb = lane >= 2 && lane < 2 + kHStripOut2 / 2 && ib < ni;
  constexpr bool SUM = MODE == kHCoeffBar;
  const bool has_mask = (MODE == kHPlain || MODE == kHVar) && A.mask != nullptr;
  const T coeff = MODE == kHPlain || MODE == kHVar ? step_coeff(A) : T(0);
  const T gs = MODE == kHPlain ? T(1) : form_sign<T>(A.form);
  const HdiffSecond<MODE, T> second(A);
  Sum2 sum{0.0, 0.0};

  const auto row_rsrc = [&](const char* base, int64_t row_bytes, int r, int rows, uint32_t width) {
    const bool in = r >= 0 && r < rows;
    return make_rsrc(base + (in ? (int64_t)r * row_bytes : 0), in ? width : 0u);
  };
  const char* ubase = reinterpret_cast<const char*>(A.u) + ((int64_t)k * A.u_sk - 2 - 2 * A.u_sj) * S;
  const char* obase = reinterpret_cast<const char*>(A.out) + (int64_t)k * A.o_sk * S;
  const PairAt uat = pair_at(ia + 2, ni + 4, true), oat = pair_at(ia, ni, owna);
  // limiter bytes: one descriptor over the whole mask (below 4 GiB), lanes
  // 0..14 the x bytes of a row, lanes 16..30 its y bytes
  const auto rm = make_rsrc(A.mask, has_mask ? (uint32_t)A.ml.total : 0u);
  const int64_t W = A.ml.words, plane_xy = (int64_t)nj * W * 8;
  const int64_t x_lev = A.ml.x_off + (int64_t)k * plane_xy, y_lev = A.ml.y_off + (int64_t)k * plane_xy;
  const int mb = lane & 15;  // the lane's byte of the strip's 15
  const bool xlane = lane < 15, ylane = lane >= 16 && lane < 31;
  const uint32_t mcol = (uint32_t)(kHStripOut2 / 8 * si + mb);
  const bool mcol_in = mcol < (uint32_t)(W * 8);
  const int bshift = 2 + 4 * mb;  // byte mb holds columns 8 mb .. 8 mb + 7: lanes 2 + 4 mb .. 5 + 4 mb
  const uint32_t ex_base = (uint32_t)(A.ml.ex_off + (int64_t)k * nj), ey_base = (uint32_t)(A.ml.ey_off + (int64_t)k * ni);

  T pa[PD], pb[PD];
  [[maybe_unused]] T p2a[MODE == kHPlain ? 1 : PD], p2b[MODE == kHPlain ? 1 : PD];
  const int r0 = j0 - 2;
  constexpr int NR = TJ + 4;
  auto issue = [&](int r, int s) {
    const auto ru = row_rsrc(ubase, A.u_sj * S, r + 2, nj + 4, (uint32_t)(ni + 4) * S);
    if constexpr (MODE != kHPlain) {
      const f32x2_t v = buf_ld2(row_rsrc(second.base + k * second.level, second.row, r - 2, second.has ? nj : 0, (uint32_t)ni * S), oat.off);
      p2a[s] = v[0];
      p2b[s] = v[1];
    }
    const f32x2_t v = buf_ld2(ru, uat.off);
    pa[s] = v[0];
    pb[s] = v[1];
  };

  T u1a = 0, u1b = 0, u2a = 0, u2b = 0, lap2a = 0, lap2b = 0, Fx2a = 0, Fx2b = 0, Fy3a = 0, Fy3b = 0;
  auto step = [&](int n, int s, bool refill) {
    const int R = r0 + n;
    T uRa = pa[s], uRb = pb[s];
    asm volatile("" : "+v"(uRa), "+v"(uRb));  // copies of their own: the slots are free for the refill
    if constexpr (ODD) {
      uRa = uat.last ? uRb : uRa;
      uRb = uat.last ? T(0) : uRb;
    }
    [[maybe_unused]] T x2a = T(0), x2b = T(0);
    if constexpr (MODE != kHPlain) {
      x2a = p2a[s];
      x2b = p2b[s];
      asm volatile("" : "+v"(x2a), "+v"(x2b));
      if constexpr (ODD) x2a = oat.last ? x2b : x2a;  // column b of that lane is not owned
    }
    if (refill) issue(R + PD, s);
    // the shifts run with every lane active (a disabled lane would read as 0)
    const T u1a_e = lane_shift<kDppWaveShl1>(u1a);  // east of b
    const T u1b_w = lane_shift<kDppWaveShr1>(u1b);  // west of a
    const T lap1a = T(4) * u1a - ((u1b_w + u1b) + (u2a + uRa));  // lap(R-1)
    const T lap1b = T(4) * u1b - ((u1a + u1a_e) + (u2b + uRb));
    const T lap1a_e = lane_shift<kDppWaveShl1>(lap1a);
    const T Fx2b_w = lane_shift<kDppWaveShr1>(Fx2b);
    const T fxa = lap1b - lap1a, fxb = lap1a_e - lap1b;  // x fluxes of row R-1
    const bool kxa = flux_kept(fxa, gs * (u1b - u1a)), kxb = flux_kept(fxb, gs * (u1a_e - u1b));
    const T Fx1a = kxa ? fxa : T(0), Fx1b = kxb ? fxb : T(0);
    const T fya = lap1a - lap2a, fyb = lap1b - lap2b;  // y fluxes between rows R-2 and R-1
    const bool kya = flux_kept(fya, gs * (u1a - u2a)), kyb = flux_kept(fyb, gs * (u1b - u2b));
    const T Fy2a = kya ? fya : T(0), Fy2b = kyb ? fyb : T(0);
    const int q = R - 2;  // out(R-2)
    const T diva = (Fx2a - Fx2b_w) + (Fy2a - Fy3a), divb = (Fx2b - Fx2a) + (Fy2b - Fy3b);
    const bool qrow = q >= j0 && q < j0 + TJ;  // uniform
    if constexpr (SUM) {
      if (qrow && q < nj) {
        sum.add_product(owna ? x2a : T(0), owna ? gs * diva : T(0));
        sum.add_product(ownb ? x2b : T(0), ownb ? gs * divb : T(0));
      }
    }
    T va, vb;
    if constexpr (MODE == kHPlain) {
      va = u2a - coeff * diva;
      vb = u2b - coeff * divb;
    } else if constexpr (MODE == kHVar) {
      va = u2a - (gs * (second.has ? x2a : coeff)) * diva;
      vb = u2b - (gs * (second.has ? x2b : coeff)) * divb;
    } else {
      va = -(x2a * (gs * diva));
      vb = -(x2b * (gs * divb));
    }
    if (!SUM && qrow) buf_st2<ODD>(row_rsrc(obase, A.o_sj * S, q, nj, (uint32_t)ni * S), oat, va, vb);
    if (has_mask) {
      const int rx = R - 1;
      const uint64_t bxa = __ballot(owna && kxa), bxb = __ballot(ownb && kxb);
      const uint64_t bya = __ballot(owna && kya), byb = __ballot(ownb && kyb);
      const bool xrow = rx >= j0 && rx < j0 + TJ && rx < nj, yrow = qrow && q < nj;  // uniform
      const uint64_t ba = ylane ? bya : bxa, bb = ylane ? byb : bxb;
      const uint8_t byte = (uint8_t)(spread4((uint32_t)(ba >> bshift) & 15u) | (spread4((uint32_t)(bb >> bshift) & 15u) << 1));
      uint32_t off = kOffNone;
      if (xlane && xrow && mcol_in) off = (uint32_t)(x_lev + (int64_t)rx * W * 8) + mcol;
      if (ylane && yrow && mcol_in) off = (uint32_t)(y_lev + (int64_t)q * W * 8) + mcol;
      buf_st_u8(rm, off, byte);
      // the x flux at i = -1 (column b of lane 1 in the first strip) and the
      // y flux below row 0 have byte planes of their own
      if (si == 0 && xrow && rx >= 0) buf_st_u8(rm, ib == -1 ? ex_base + (uint32_t)rx : kOffNone, kxb ? 1 : 0);
      if (q == -1) {
        buf_st_u8(rm, owna ? ey_base + (uint32_t)ia : kOffNone, kya ? 1 : 0);
        buf_st_u8(rm, ownb ? ey_base + (uint32_t)ib : kOffNone, kyb ? 1 : 0);
      }
    }
    Fy3a = Fy2a; Fy3b = Fy2b;
    Fx2a = Fx1a; Fx2b = Fx1b;
    lap2a = lap1a; lap2b = lap1b;
    u2a = u1a; u2b = u1b;
    u1a = uRa; u1b = uRb;
  };

#pragma unroll
  for (int s = 0; s < PD; ++s) issue(r0 + s, s);
  int n = 0;
  for (; n < NR - PD; n += PD) {
#pragma unroll
    for (int s = 0; s < PD; ++s) step(n + s, s, true);
  }
#pragma unroll
  for (int s = 0; s < PD; ++s) step(n + s, s, false);
  if constexpr (MODE == kHPlain || MODE == kHVar) keep_coeff(A, coeff, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6));
  return sum;
}

// LANE: columns per lane, 1, 2 (FP32, even ni) or 3: two with odd ni.
template <typename T, int MODE, int LANE>
__device__ __forceinline__ Sum2 hdiff_strip_of(const StepArgs<T>& A, int t, int k) {
    using H = HStrip<MODE, LANE>;
  if constexpr (LANE > 1) return hdiff_strip2<H::rows, H::pd, MODE, LANE == 3>(A, t, k);
  else return hdiff_strip<T, H::rows, H::pd, MODE>(A, t, k);
}

// One strip per wave, at one level per grid row.
template <typename T, int MODE, int LANE>
__global__ void __launch_bounds__(kWG) k_hdiff_strip(StepArgs<T> A) {
  // the wave's strip (uniform: the conditions on it stay scalar branches)
  const int t = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * kStripsPerWG +
                                               (int)(threadIdx.x >> 6));
  if (t >= A.ntiles) return;  // whole waves only: no barrier follows
  hdiff_strip_of<T, MODE, LANE>(A, t, blockIdx.y);
}

// strips of the walk in i and in all
template <typename T, int MODE, int LANE>
inline void hdiff_strip_count(StepArgs<T>& A) {
  constexpr int W = LANE > 1 ? kHStripOut2 : kHStripOut, R = HStrip<MODE, LANE>::rows;
  A.tiles_i = (A.ni + W - 1) / W;
  A.ntiles = A.tiles_i * ((A.nj + R - 1) / R);
}

// calls go(LANE) for the domain
template <typename T, typename F>
inline void hdiff_strip_lanes(const StepArgs<T>& A, F&& go) {
  if constexpr (sizeof(T) == 4) {
    if (A.ni > 1 && A.ni % 2 == 0) return go(std::integral_constant<int, 2>{});
    if (A.ni > 1) return go(std::integral_constant<int, 3>{});
  }
  go(std::integral_constant<int, 1>{});
}

template <typename T, int MODE>
hipError_t launch_hdiff_strip(StepArgs<T> A, hipStream_t s) {
  hdiff_strip_lanes(A, [&](auto lane) {
    constexpr int L = decltype(lane)::value;
    hdiff_strip_count<T, MODE, L>(A);
    const dim3 grid((A.ntiles + kStripsPerWG - 1) / kStripsPerWG, A.nk), block(kWG);
    hipLaunchKernelGGL((k_hdiff_strip<T, MODE, L>), grid, block, 0, s, A);
  });
  return hipGetLastError();
}

// grid.y's documented limit: the walk has one grid row per level
constexpr int kMaxGridY = 65535;

}  // namespace gt4mi
