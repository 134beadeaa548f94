// api.cpp -- the C ABI (include/stencil.h): O(1) host-side validation of
// field metadata, implementation choice and kernel dispatch.  No call reads
// device memory, allocates or synchronises (the autotuner excepted).
#include <hip/hip_runtime.h>

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/stencil.h"
#include "api_internal.hpp"
#include "common.hpp"
#include "launch.hpp"

namespace gt4mi {

// ------------------------------------------------------------------ errors
static thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int ok() { return STENCIL_OK; }

int hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return STENCIL_OK;
  return fail(STENCIL_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

// ------------------------------------------------------------------ device
// The kernels are compiled for gfx950 only; refuse other devices up front.
int check_device() {
  static std::mutex mu;
  static std::vector<int> known;  // per device: 0 unknown, 1 ok, -1 unsupported
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_status(e, "hipGetDevice");
  std::lock_guard<std::mutex> lk(mu);
  if ((int)known.size() <= dev) known.resize(dev + 1, 0);
  if (known[dev] == 0) {
    hipDeviceProp_t p;
    e = hipGetDeviceProperties(&p, dev);
    if (e != hipSuccess) return hip_status(e, "hipGetDeviceProperties");
    known[dev] = (strncmp(p.gcnArchName, "gfx950", 6) == 0) ? 1 : -1;
    if (known[dev] < 0)
      return fail(STENCIL_E_UNSUPPORTED, "device %d is %s; this library is built for gfx950", dev,
                  p.gcnArchName);
  }
  if (known[dev] < 0) return fail(STENCIL_E_UNSUPPORTED, "device %d is not gfx950", dev);
  return STENCIL_OK;
}

// ------------------------------------------------------------------ validation
size_t esize(stencil_dtype dt) { return dt == STENCIL_F64 ? 8 : 4; }

int check_dtype(stencil_dtype dt) {
  if (dt != STENCIL_F32 && dt != STENCIL_F64) return fail(STENCIL_E_DTYPE, "unknown dtype %d", (int)dt);
  return STENCIL_OK;
}

static const int64_t kMaxExtent = int64_t(1) << 31;

int check_domain(const int64_t* dom) {
  if (!dom) return fail(STENCIL_E_NULL, "domain is NULL");
  for (int d = 0; d < 3; ++d)
    if (dom[d] < 0 || dom[d] >= kMaxExtent)
      return fail(STENCIL_E_SHAPE, "domain[%d] = %lld out of range", d, (long long)dom[d]);
  return STENCIL_OK;
}

bool domain_empty(const int64_t* dom) { return dom[0] == 0 || dom[1] == 0 || dom[2] == 0; }

// Byte range [lo, hi) spanned by a field's allocation.
Span span_of(const stencil_field* f, size_t es) {
  Span s;
  s.lo = reinterpret_cast<uintptr_t>(f->data);
  int64_t last = 0;
  for (int d = 0; d < 3; ++d) last += (f->shape[d] > 0 ? f->shape[d] - 1 : 0) * f->stride[d];
  s.hi = s.lo + (uintptr_t)(last + 1) * es;
  return s;
}

bool overlap(Span a, Span b) { return a.lo < b.hi && b.lo < a.hi; }

int check_field(const char* name, const stencil_field* f, const int64_t* dom, Role role, size_t es) {
  if (!f) return fail(STENCIL_E_NULL, "%s: field is NULL", name);
  if (!f->data) return fail(STENCIL_E_NULL, "%s.data is NULL", name);
  if (reinterpret_cast<uintptr_t>(f->data) % es)
    return fail(STENCIL_E_DTYPE, "%s.data is not aligned to %zu bytes", name, es);
  for (int d = 0; d < 3; ++d) {
    if (f->shape[d] < 0 || f->shape[d] >= kMaxExtent)
      return fail(STENCIL_E_SHAPE, "%s.shape[%d] = %lld out of range", name, d, (long long)f->shape[d]);
    if (f->origin[d] < 0 || f->origin[d] >= kMaxExtent)
      return fail(STENCIL_E_SHAPE, "%s.origin[%d] = %lld out of range", name, d, (long long)f->origin[d]);
  }
  if (f->stride[0] != 1) return fail(STENCIL_E_STRIDE, "%s.stride[0] = %lld, must be 1", name, (long long)f->stride[0]);
  if (f->stride[1] < f->shape[0] || f->stride[1] >= (int64_t(1) << 40))
    return fail(STENCIL_E_STRIDE, "%s.stride[1] = %lld overlaps rows (shape[0] = %lld)", name,
                (long long)f->stride[1], (long long)f->shape[0]);
  if (f->stride[2] < f->stride[1] * f->shape[1] || f->stride[2] >= (int64_t(1) << 46))
    return fail(STENCIL_E_STRIDE, "%s.stride[2] = %lld overlaps planes", name, (long long)f->stride[2]);
  // kernels address within a level with 32-bit byte offsets, and predicate a
  // lane's access off with the offset kOffNone, which must stay outside every
  // window: a level may span at most kOffNone - 16 bytes
  if ((f->stride[1] * f->shape[1] + f->shape[0]) * (int64_t)es > (int64_t)kOffNone - 16)
    return fail(STENCIL_E_UNSUPPORTED, "%s: one level spans %lld bytes, above the 32-bit window limit %lld", name,
                (long long)((f->stride[1] * f->shape[1] + f->shape[0]) * (int64_t)es),
                (long long)((int64_t)kOffNone - 16));
  const int64_t h = (role == ROLE_HALO) ? kHalo : 0;
  for (int d = 0; d < 2; ++d) {
    if (f->origin[d] < h)
      return fail(STENCIL_E_HALO, "%s.origin[%d] = %lld leaves no room for the %lld-point halo", name,
                  d, (long long)f->origin[d], (long long)h);
    if (f->origin[d] + dom[d] + h > f->shape[d])
      return fail(h ? STENCIL_E_HALO : STENCIL_E_SHAPE,
                  "%s: origin[%d] + domain[%d] (+ halo %lld) = %lld exceeds shape %lld", name, d, d,
                  (long long)h, (long long)(f->origin[d] + dom[d] + h), (long long)f->shape[d]);
  }
  const int64_t kext = dom[2] + (role == ROLE_STAGGERED ? 1 : 0);
  if (f->origin[2] + kext > f->shape[2])
    return fail(STENCIL_E_SHAPE, "%s: origin[2] + %lld levels = %lld exceeds shape[2] = %lld", name,
                (long long)kext, (long long)(f->origin[2] + kext), (long long)f->shape[2]);
  return STENCIL_OK;
}

int check_no_alias(const char* oname, Span o, const char* iname, Span in) {
  if (overlap(o, in)) return fail(STENCIL_E_ALIAS, "%s overlaps %s", oname, iname);
  return STENCIL_OK;
}

// ------------------------------------------------------------------ options
// Whether a 128-column tile can run: the fused two-ended step only.
static bool narrow_tile_runs(const ResolvedOpts& r, int op, stencil_dtype dt, const int64_t* dom) {
  return op == STENCIL_OP_STEP && r.impl != STENCIL_IMPL_PLAIN && r.column_store == STENCIL_COLUMN_SPLIT &&
         dom[2] <= split_step_limit((int)esize(dt));
}

// The two-ended step's tile where nothing chose one, from 230 sizes of 8 to 144
// levels in four forms (plain, mask, coefficient field, damping), each with fields
// that stay in the last-level cache from call to call and with three sets in turn.
// While the step's four fields fit half that cache, a level costs its instructions,
// not its bytes: tiles of 128 columns spread them over twice the workgroups (one wave
// per SIMD each where the chip is not full) and, in FP64, 16-wide rows load the box in
// two passes instead of three.  64x4 against 16x8 (FP64) and 32x4 (FP32), us: FP64
// 39x89x29 11.9, 8.3, 128x128x80 28.5, 20.0; FP32 39x89x29 9.2, 8.0, 256x200x80 22.4,
// 20.6, 256x256x80 22.9, 21.1.  Not where 64x4 fills the chip by itself: FP32 of more
// than a workgroup per CU and a quarter of the cache (three sets 771x141x61 28.2,
// 32.6, 491x238x56 27.9, 32.9, 512x512x20 20.1, 22.2; one set the same or 5% less),
// FP64 of one round of 64x4 where 16x8 tiles are more than 256 and the fields 0.4 of
// the cache, or the tiles more than three to a CU, which take 32x8 (three sets, 64x4,
// 16x8, 32x8: 256x200x80 33.3, 39.3, 31.8, 626x90x73 33.3, 39.9, 32.6; one set 0.90 to
// 0.97 and 0.95 of 64x4; 800 tiles 512x200x32 25.9, 31.4, 26.1, one set 20.6, 22.7,
// 20.2; but 494 tiles 200x300x30 19.8, 13.2, 18.4, one set 19.6, 13.1, 18.2, 760 tiles
// 300x320x30 22.9, 20.8, 22.1, one set 20.1, 17.3, 19.0), or 64x4 in the long class of
// the generalised step (763x42x113 65.6, 88.5; 626x59x107 70.7, 88.0).
// Past half the cache (other buffers of the program share it) 64x4 loses where it
// leaves places for workgroups idle, a tenth of them where a CU holds one workgroup:
// 64x4 against 32x4, FP64 501x403x60 107, 98.6 (with mask 113, 104), 400x300x60 66.9,
// 48.9, 384x384x64 79.5, 73.0, 400x256x100 104, 99.4; FP32 512x300x90 68.8, 52.4.  In
// FP32 with just two rounds it depends on the cache: 400x256x100 one set 48.5, 41.7,
// three 52.3, 57.4.  Where a CU holds two, the other keeps it busy until a quarter is
// idle: FP32 400x300x60 35.3, 25.6, FP64 512x300x32 36.2, 32.4, but FP32 512x400x80,
// 22% idle, 58.9, 60.7.  With whole rounds 32x8 is faster in FP64 while the fields fit
// the cache (256x256x80 32.4 to 34.2, 30.6; the generalised step not: 512x512x28
// 69.5, 71.2) and 64x4 streams best elsewhere (against 32x4: FP64 512x256x80 74.6,
// 78.3, 512x512x80 151.4, 152.5; FP32 512x256x80 33.4, 38.2, 512x512x80 77.9, 89.1).
// FP64 columns of the generalised step that spill with 128 columns keep 64x4: 81 to 96
// levels (512x300x90 155, 173), and longer ones on large domains (400x256x100 144,
// 158; but 60x60x110 71.3, 55.5 and 200x200x100 78.5, 76.7 with 16x8).  The long FP64
// class runs tiles of 128 columns one to a CU whatever the width: no other where 64x2
// takes fewer rounds (763x42x113 32.5, 16x8 52.9).
constexpr int64_t kLastLevelCache = int64_t(256) << 20;
static void default_step_tile(ResolvedOpts& r, stencil_dtype dt, const int64_t* dom, bool variant) {
  const int64_t es = (int64_t)esize(dt), nk = dom[2], bytes = 4 * es * dom[0] * dom[1] * nk;
  const bool f64 = es == 8;
  bool small = 2 * bytes <= kLastLevelCache;
  if (f64 && variant && nk > 80 && (nk <= kSplitRegNkF64 || !small)) return;
  auto tiles = [&](int ti, int tj) { return ((dom[0] + ti - 1) / ti) * ((dom[1] + tj - 1) / tj); };
  const int64_t n = tiles(64, 4), per_cu = split_tiles_per_cu((int)es, nk), slots = kCus * per_cu;
  const int64_t places = (n + slots - 1) / slots * slots;
  if (!f64) small = small && (n <= kCus || 4 * bytes <= kLastLevelCache || (per_cu == 3 && n <= slots));
  const bool idle = per_cu < 3 && (per_cu == 1 ? 10 : 4) * (places - n) >= places;
  int ti = 64, tj = 4;
  if (small || idle) ti = f64 && small ? 16 : 32, tj = 128 / ti;
  else if (f64 && !variant && bytes <= kLastLevelCache) ti = 32, tj = 8;
  if (f64 && nk > kSplitRegNkF64 && !variant) {
    auto rounds = [&](int w) { return (tiles(w, kSplitLongNT / w) + kCus - 1) / kCus; };
    if (rounds(ti) > rounds(64)) ti = 64, tj = 4;
  } else if (ti == 16 && n <= slots && tiles(16, 8) > kCus) {
    if (nk > kSplitRegNkF64) ti = 64, tj = 4;
    else if (tiles(16, 8) > 3 * kCus || 5 * bytes > 2 * kLastLevelCache) ti = 32, tj = 8;
  }
  r.tile_i = ti;
  r.tile_j = tj;
}

ResolvedOpts resolve_opts(const stencil_options* o, stencil_dtype dt, int op, const int64_t* dom) {
  ResolvedOpts r;
  r.impl = o ? o->impl : STENCIL_IMPL_AUTO;
  int32_t ti = 0, tj = 0, col = 0, ord = 0;
  const bool tuned = tuning_get(dt, op, dom, &ti, &tj, &col, &ord);
  const bool own_tile = o && o->tile_i;
  r.tile_i = own_tile ? o->tile_i : ti;
  r.tile_j = own_tile ? (o->tile_j ? o->tile_j : kWG / o->tile_i) : tj;
  r.column_store = (o && o->column_store) ? o->column_store : col;
  if (r.column_store == STENCIL_COLUMN_AUTO) {
    if (op == STENCIL_OP_STEP && dom[2] <= split_step_limit((int)esize(dt)))
      r.column_store = STENCIL_COLUMN_SPLIT;
    else
      r.column_store = (dt == STENCIL_F64 && dom[2] > 96) ? STENCIL_COLUMN_OUTBUF : STENCIL_COLUMN_REGISTERS;
  }
  // a tuned 128-column tile where the call does not run the two-ended step
  // (another column store, or columns past its limit) takes the 256-column
  // tile of the same width; a caller's own such tile is refused by the step
  if (!own_tile && !narrow_tile_runs(r, op, dt, dom)) r.tile_j = kWG / r.tile_i;
  if (!own_tile && !tuned && narrow_tile_runs(r, op, dt, dom)) default_step_tile(r, dt, dom, variant_opts(o));
  r.ws = o ? o->workspace : nullptr;
  r.ws_bytes = o ? o->workspace_bytes : 0;
  r.form = o ? o->hdiff_form : STENCIL_HDIFF_STATED;
  r.kappa = o ? o->coeff_field : nullptr;
  r.order = (o && o->tile_order) ? o->tile_order : ord;
  if (r.order != STENCIL_ORDER_DISPATCH) r.order = STENCIL_ORDER_XCD;
  r.dev = nullptr;
  r.wrapped = false;
  return r;
}

int check_opts(const stencil_options* o) {
  if (!o) return STENCIL_OK;
  if (o->impl < STENCIL_IMPL_AUTO || o->impl > STENCIL_IMPL_PLAIN)
    return fail(STENCIL_E_ARG, "options.impl = %d unknown", (int)o->impl);
  if (o->tile_i != 0 && !(o->tile_j == 0 && (o->tile_i == 64 || o->tile_i == 32 || o->tile_i == 16)) &&
      !tile_wide(o->tile_i, o->tile_j) && !tile_narrow(o->tile_i, o->tile_j))
    return fail(STENCIL_E_ARG, "options tile %dx%d unsupported (64x4, 32x8, 16x16; 64x2, 32x4, 16x8)",
                (int)o->tile_i, (int)o->tile_j);
  if (o->column_store < 0 || o->column_store > STENCIL_COLUMN_SPLIT)
    return fail(STENCIL_E_ARG, "options.column_store = %d unknown", (int)o->column_store);
  if (o->workspace_bytes && !o->workspace) return fail(STENCIL_E_NULL, "options.workspace is NULL");
  if (o->boundary != STENCIL_BOUNDARY_FROZEN && o->boundary != STENCIL_BOUNDARY_PERIODIC)
    return fail(STENCIL_E_ARG, "options.boundary = %d unknown", (int)o->boundary);
  if (o->hdiff_form != STENCIL_HDIFF_STATED && o->hdiff_form != STENCIL_HDIFF_DAMPING)
    return fail(STENCIL_E_ARG, "options.hdiff_form = %d unknown", (int)o->hdiff_form);
  if (o->tile_order < STENCIL_ORDER_AUTO || o->tile_order > STENCIL_ORDER_DISPATCH)
    return fail(STENCIL_E_ARG, "options.tile_order = %d unknown", (int)o->tile_order);
  return STENCIL_OK;
}

int check_coeff_field(const stencil_options* o, const int64_t* dom, size_t es, const char* oname, Span out) {
  if (!o || !o->coeff_field) return STENCIL_OK;
  TRY(check_field("coeff_field", o->coeff_field, dom, ROLE_INTERIOR, es));
  return check_no_alias(oname, out, "coeff_field", span_of(o->coeff_field, es));
}

// The generalised diffusion in the forward argument block.
template <typename T>
static void apply_variant(StepArgs<T>& A, const ResolvedOpts& r) {
  A.form = r.form;
  if (r.dev) {
    A.coeff_bytes = r.dev->f64 ? 8 : 4;
    A.c_sj = (int64_t)reinterpret_cast<uintptr_t>(r.dev->p);
    A.c_sk = (int64_t)reinterpret_cast<uintptr_t>(r.dev->copy);
  }
  if (r.kappa) {
    A.kappa = at_origin<T>(r.kappa);
    A.c_sj = r.kappa->stride[1];
    A.c_sk = r.kappa->stride[2];
  }
}

// ... and in the adjoint's: a scalar coefficient takes the form's sign
// (the damping form is the stated one with the coefficient negated, its
// saved mask already holding the damping decisions); a coefficient field
// leaves the sign in coeff.
template <typename T>
static void apply_variant(AdjArgs<T>& A, const ResolvedOpts& r, double coeff) {
  const double sg = r.form == STENCIL_HDIFF_DAMPING ? -1.0 : 1.0;
  if (r.kappa) {
    A.kappa = at_origin<T>(r.kappa);
    A.c_sj = r.kappa->stride[1];
    A.c_sk = r.kappa->stride[2];
    A.coeff = (T)sg;
  } else if (r.dev) {
    A.coeff = (T)sg;
    A.coeff_in_memory = 1;
    A.c_sj = (int64_t)reinterpret_cast<uintptr_t>(r.dev->p);
  } else {
    A.coeff = (T)(sg * coeff);
  }
}

// Plain-form workspace carve-up: lap, fx, fy, c', d' (each 256-B aligned).
static int64_t r256(int64_t b) { return (b + 255) & ~int64_t(255); }

size_t plain_ws_bytes(size_t es, const int64_t* dom) {
  const int64_t ni = dom[0], nj = dom[1], nk = dom[2];
  return (size_t)(r256((ni + 2) * (nj + 2) * nk * es) + r256((ni + 1) * nj * nk * es) +
                  r256(ni * (nj + 1) * nk * es) + 2 * r256(ni * nj * nk * es));
}

template <typename T>
PlainWs<T> carve_plain(void* ws, const int64_t* dom) {
  const int64_t ni = dom[0], nj = dom[1], nk = dom[2];
  const int64_t es = sizeof(T);
  char* p = static_cast<char*>(ws);
  PlainWs<T> w;
  w.lap = reinterpret_cast<T*>(p);
  p += r256((ni + 2) * (nj + 2) * nk * es);
  w.fx = reinterpret_cast<T*>(p);
  p += r256((ni + 1) * nj * nk * es);
  w.fy = reinterpret_cast<T*>(p);
  p += r256(ni * (nj + 1) * nk * es);
  w.cp = reinterpret_cast<T*>(p);
  p += r256(ni * nj * nk * es);
  w.dp = reinterpret_cast<T*>(p);
  return w;
}

// column-adjoint workspace: lambda (when data_bar is absent) then y and c'
size_t adj_ws_bytes(size_t es, const int64_t* dom, bool need_lam, bool plain) {
  const int64_t n = dom[0] * dom[1] * dom[2];
  return (size_t)((need_lam ? r256(n * es) : 0) + (plain ? 2 * r256(n * es) : 0));
}

// ------------------------------------------------------------------ arg blocks
template <typename T>
StepArgs<T> step_args(const stencil_field* u, const stencil_field* data, const stencil_field* w,
                      stencil_field* out, const int64_t* dom, double coeff, double dt_dz,
                      void* mask) {
  StepArgs<T> A;
  memset(&A, 0, sizeof A);
  if (u) { A.u = at_origin<T>(u); A.u_sj = u->stride[1]; A.u_sk = u->stride[2]; }
  if (data) { A.data = at_origin<T>(data); A.d_sj = data->stride[1]; A.d_sk = data->stride[2]; }
  if (w) { A.w = at_origin<T>(w); A.w_sj = w->stride[1]; A.w_sk = w->stride[2]; }
  if (out) { A.out = at_origin_mut<T>(out); A.o_sj = out->stride[1]; A.o_sk = out->stride[2]; }
  A.mask = static_cast<uint8_t*>(mask);
  A.ml = MaskLayout::make(dom[0], dom[1], dom[2]);
  A.ni = (int)dom[0];
  A.nj = (int)dom[1];
  A.nk = (int)dom[2];
  A.coeff = (T)coeff;
  A.r4 = (T)(0.25 * dt_dz);
  return A;
}

template StepArgs<float> step_args<float>(const stencil_field*, const stencil_field*, const stencil_field*,
                                          stencil_field*, const int64_t*, double, double, void*);
template StepArgs<double> step_args<double>(const stencil_field*, const stencil_field*, const stencil_field*,
                                            stencil_field*, const int64_t*, double, double, void*);

template <typename T>
AdjArgs<T> adj_args(const stencil_field* xbar, const stencil_field* w, T* lam, int64_t l_sj,
                    int64_t l_sk, stencil_field* ubar, const int64_t* dom, double coeff,
                    double dt_dz, const void* mask) {
  AdjArgs<T> A;
  memset(&A, 0, sizeof A);
  if (xbar) { A.xbar = at_origin<T>(xbar); A.x_sj = xbar->stride[1]; A.x_sk = xbar->stride[2]; }
  if (w) { A.w = at_origin<T>(w); A.w_sj = w->stride[1]; A.w_sk = w->stride[2]; }
  A.lam = lam;
  A.l_sj = l_sj;
  A.l_sk = l_sk;
  if (ubar) { A.ubar = at_origin_mut<T>(ubar); A.b_sj = ubar->stride[1]; A.b_sk = ubar->stride[2]; }
  A.mask = static_cast<const uint8_t*>(mask);
  A.ml = MaskLayout::make(dom[0], dom[1], dom[2]);
  A.ni = (int)dom[0];
  A.nj = (int)dom[1];
  A.nk = (int)dom[2];
  A.coeff = (T)coeff;
  A.r4 = (T)(0.25 * dt_dz);
  return A;
}

template AdjArgs<float> adj_args<float>(const stencil_field*, const stencil_field*, float*, int64_t, int64_t,
                                      stencil_field*, const int64_t*, double, double, const void*);
template AdjArgs<double> adj_args<double>(const stencil_field*, const stencil_field*, double*, int64_t, int64_t,
                                        stencil_field*, const int64_t*, double, double, const void*);

// ------------------------------------------------------------------ dispatch
template <typename T>
int run_hdiff(const stencil_field* u, stencil_field* out, const int64_t* dom, double coeff,
              void* mask, const ResolvedOpts& r, hipStream_t s) {
  StepArgs<T> A = step_args<T>(u, nullptr, nullptr, out, dom, coeff, 0.0, mask);
  if (r.impl == STENCIL_IMPL_PLAIN)
    return hip_status(launch_hdiff_plain<T>(A, carve_plain<T>(r.ws, dom), s), "hdiff (plain)");
  apply_variant(A, r);
  return hip_status(launch_hdiff_fused<T>(A, r.tile_i, s), "hdiff (fused)");
}

template <typename T>
int run_vadv(const stencil_field* u, const stencil_field* data, const stencil_field* w,
             stencil_field* out, const int64_t* dom, double dt_dz, const ResolvedOpts& r,
             hipStream_t s) {
  StepArgs<T> A = step_args<T>(u, data, w, out, dom, 0.0, dt_dz, nullptr);
  if (r.impl == STENCIL_IMPL_PLAIN)
    return hip_status(launch_vadv_plain<T>(A, carve_plain<T>(r.ws, dom), s), "vadv (plain)");
  return hip_status(launch_vadv_fused<T>(A, s), "vadv (fused)");
}

template <typename T>
int run_step(const stencil_field* u, const stencil_field* data, const stencil_field* w,
             stencil_field* out, const int64_t* dom, double coeff, double dt_dz, void* mask,
             const ResolvedOpts& r, hipStream_t s) {
  if (r.impl == STENCIL_IMPL_PLAIN) {
    PlainWs<T> ws = carve_plain<T>(r.ws, dom);
    StepArgs<T> A = step_args<T>(u, nullptr, nullptr, out, dom, coeff, 0.0, mask);
    int rc = hip_status(launch_hdiff_plain<T>(A, ws, s), "step (plain hdiff)");
    if (rc) return rc;
    // the diffused field now sits in out's interior: it is the u_k of d_k
    StepArgs<T> B = step_args<T>(out, data, w, out, dom, coeff, dt_dz, nullptr);
    return hip_status(launch_vadv_plain<T>(B, ws, s), "step (plain vadv)");
  }
  StepArgs<T> A = step_args<T>(u, data, w, out, dom, coeff, dt_dz, mask);
  apply_variant(A, r);
  A.order = r.order;
  A.wrapped = r.wrapped;
  return hip_status(launch_step_fused<T>(A, r.tile_i, r.tile_j, r.column_store, s), "step (fused)");
}

template <typename T>
int run_hdiff_adjoint(const T* lam, int64_t l_sj, int64_t l_sk, const void* mask,
                      stencil_field* ubar, const int64_t* dom, double coeff, const ResolvedOpts& r,
                      hipStream_t s) {
  AdjArgs<T> A = adj_args<T>(nullptr, nullptr, const_cast<T*>(lam), l_sj, l_sk, ubar, dom, coeff,
                             0.0, (dom[0] == 0 || dom[1] == 0) ? nullptr : mask);
  apply_variant(A, r, coeff);
  return hip_status(launch_hdiff_adjoint<T>(A, s), "hdiff adjoint");
}

template <typename T>
int run_vadv_adjoint(const stencil_field* xbar, const stencil_field* w, T* lam, int64_t l_sj,
                     int64_t l_sk, const int64_t* dom, double dt_dz, const ResolvedOpts& r,
                     void* ws_after_lam, hipStream_t s) {
  AdjArgs<T> A = adj_args<T>(xbar, w, lam, l_sj, l_sk, nullptr, dom, 0.0, dt_dz, nullptr);
  const bool plain = r.impl == STENCIL_IMPL_PLAIN || dom[2] > kMaxFusedNk;
  T* y = nullptr;
  T* c = nullptr;
  if (plain) {
    const int64_t n = dom[0] * dom[1] * dom[2];
    y = static_cast<T*>(ws_after_lam);
    c = reinterpret_cast<T*>(static_cast<char*>(ws_after_lam) + r256(n * (int64_t)sizeof(T)));
  }
  return hip_status(launch_vadv_adjoint<T>(A, plain ? 1 : 0, y, c, s), "vadv adjoint");
}

}  // namespace gt4mi

using namespace gt4mi;

// ====================================================================== C ABI
extern "C" {

int stencil_version(void) { return STENCIL_ABI_VERSION; }

const char* stencil_last_error(void) { return g_err.c_str(); }

int stencil_max_fused_nk(stencil_dtype dtype) {
  (void)dtype;
  return kMaxFusedNk;
}

size_t stencil_mask_bytes(const int64_t domain[3]) {
  if (!domain) return 0;
  for (int d = 0; d < 3; ++d)
    if (domain[d] < 0 || domain[d] >= kMaxExtent) return 0;
  return (size_t)MaskLayout::make(domain[0], domain[1], domain[2]).total;
}

size_t stencil_workspace_bytes(int op, stencil_dtype dtype, const int64_t domain[3],
                               const stencil_options* opts) {
  if (check_dtype(dtype) || check_domain(domain)) return 0;
  const size_t es = esize(dtype);
  const bool plain = (opts && opts->impl == STENCIL_IMPL_PLAIN) || domain[2] > kMaxFusedNk;
  switch (op) {
    case STENCIL_OP_HDIFF:
    case STENCIL_OP_VADV:
    case STENCIL_OP_STEP:
      return plain ? plain_ws_bytes(es, domain) : 0;
    case STENCIL_OP_HDIFF_ADJOINT:
      return 0;
    case STENCIL_OP_VADV_ADJOINT:
      return adj_ws_bytes(es, domain, false, plain);
    case STENCIL_OP_STEP_ADJOINT:
      return adj_ws_bytes(es, domain, true, plain);
    default:
      return 0;
  }
}

static int need_plain_ws(const ResolvedOpts& r, size_t need) {
  if (need == 0) return STENCIL_OK;
  if (!r.ws) return fail(STENCIL_E_WORKSPACE, "this call needs %zu bytes of workspace (options.workspace is NULL)", need);
  if (r.ws_bytes < need)
    return fail(STENCIL_E_WORKSPACE, "workspace of %zu bytes is smaller than the %zu needed", r.ws_bytes, need);
  return STENCIL_OK;
}

static int fused_nk_ok(ResolvedOpts& r, const int64_t* dom) {
  if (r.impl == STENCIL_IMPL_PLAIN) return STENCIL_OK;
  if (dom[2] > kMaxFusedNk) {
    if (r.impl == STENCIL_IMPL_FUSED)
      return fail(STENCIL_E_UNSUPPORTED, "nk = %lld exceeds the fused column limit %d; use STENCIL_IMPL_PLAIN",
                  (long long)dom[2], kMaxFusedNk);
    r.impl = STENCIL_IMPL_PLAIN;
  }
  return STENCIL_OK;
}

static int hdiff_call(stencil_dtype dtype, const stencil_field* u, stencil_field* out,
                  const int64_t domain[3], double coeff, void* mask, const stencil_options* opts,
                  hipStream_t stream,
                  const DevCoeff* dev) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  TRY(check_opts(opts));
  const size_t es = esize(dtype);
  TRY(check_field("u", u, domain, ROLE_HALO, es));
  TRY(check_field("out", out, domain, ROLE_INTERIOR, es));
  TRY(check_no_alias("out", span_of(out, es), "u", span_of(u, es)));
  TRY(check_coeff_field(opts, domain, es, "out", span_of(out, es)));
  if (mask) {
    Span m{reinterpret_cast<uintptr_t>(mask), reinterpret_cast<uintptr_t>(mask) + stencil_mask_bytes(domain)};
    TRY(check_no_alias("mask", m, "u", span_of(u, es)));
    TRY(check_no_alias("mask", m, "out", span_of(out, es)));
    if (opts && opts->coeff_field) TRY(check_no_alias("mask", m, "coeff_field", span_of(opts->coeff_field, es)));
  }
  if (domain_empty(domain)) return ok();
  ResolvedOpts r = resolve_opts(opts, dtype, STENCIL_OP_HDIFF, domain);
  r.dev = dev;
  if (variant_opts(opts) && r.impl == STENCIL_IMPL_PLAIN)
    return fail(STENCIL_E_UNSUPPORTED, "the generalised diffusion runs the fused kernels only");
  if (r.impl == STENCIL_IMPL_PLAIN) TRY(need_plain_ws(r, plain_ws_bytes(es, domain)));
  TRY(check_device());
  return dtype == STENCIL_F64 ? run_hdiff<double>(u, out, domain, coeff, mask, r, stream)
                              : run_hdiff<float>(u, out, domain, coeff, mask, r, stream);
}

int stencil_hdiff(stencil_dtype dtype, const stencil_field* u, stencil_field* out,
                  const int64_t domain[3], double coeff, void* mask, const stencil_options* opts,
                  hipStream_t stream) {
  return hdiff_call(dtype, u, out, domain, coeff, mask, opts, stream, nullptr);
}

int stencil_vadv(stencil_dtype dtype, const stencil_field* u, const stencil_field* data,
                 const stencil_field* w, stencil_field* out, const int64_t domain[3], double dt_dz,
                 const stencil_options* opts, hipStream_t stream) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  TRY(check_opts(opts));
  const size_t es = esize(dtype);
  TRY(check_field("u", u, domain, ROLE_INTERIOR, es));
  TRY(check_field("data", data, domain, ROLE_INTERIOR, es));
  TRY(check_field("w", w, domain, ROLE_STAGGERED, es));
  const bool periodic = opts && opts->boundary == STENCIL_BOUNDARY_PERIODIC;
  TRY(check_field("out", out, domain, periodic ? ROLE_HALO : ROLE_INTERIOR, es));
  const Span so = span_of(out, es);
  TRY(check_no_alias("out", so, "u", span_of(u, es)));
  TRY(check_no_alias("out", so, "data", span_of(data, es)));
  TRY(check_no_alias("out", so, "w", span_of(w, es)));
  if (domain_empty(domain)) return ok();
  ResolvedOpts r = resolve_opts(opts, dtype, STENCIL_OP_VADV, domain);
  TRY(fused_nk_ok(r, domain));
  if (r.impl == STENCIL_IMPL_PLAIN) TRY(need_plain_ws(r, plain_ws_bytes(es, domain)));
  TRY(check_device());
  return dtype == STENCIL_F64 ? run_vadv<double>(u, data, w, out, domain, dt_dz, r, stream)
                              : run_vadv<float>(u, data, w, out, domain, dt_dz, r, stream);
}

static int step_call(stencil_dtype dtype, const stencil_field* u, const stencil_field* data,
                 const stencil_field* w, stencil_field* out, const int64_t domain[3], double coeff,
                 double dt_dz, void* mask, const stencil_options* opts, hipStream_t stream,
                  const DevCoeff* dev, const LoopPlan* loop = nullptr, bool wrapped = false) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  TRY(check_opts(opts));
  const size_t es = esize(dtype);
  TRY(check_field("u", u, domain, ROLE_HALO, es));
  TRY(check_field("data", data, domain, ROLE_INTERIOR, es));
  TRY(check_field("w", w, domain, ROLE_STAGGERED, es));
  const bool periodic = opts && opts->boundary == STENCIL_BOUNDARY_PERIODIC;
  TRY(check_field("out", out, domain, periodic ? ROLE_HALO : ROLE_INTERIOR, es));
  const Span so = span_of(out, es);
  TRY(check_no_alias("out", so, "u", span_of(u, es)));
  TRY(check_no_alias("out", so, "data", span_of(data, es)));
  TRY(check_no_alias("out", so, "w", span_of(w, es)));
  if (mask) {
    Span m{reinterpret_cast<uintptr_t>(mask), reinterpret_cast<uintptr_t>(mask) + stencil_mask_bytes(domain)};
    TRY(check_no_alias("mask", m, "u", span_of(u, es)));
    TRY(check_no_alias("mask", m, "out", so));
    TRY(check_no_alias("mask", m, "data", span_of(data, es)));
    TRY(check_no_alias("mask", m, "w", span_of(w, es)));
    if (opts && opts->coeff_field) TRY(check_no_alias("mask", m, "coeff_field", span_of(opts->coeff_field, es)));
  }
  TRY(check_coeff_field(opts, domain, es, "out", so));
  if (domain_empty(domain)) return ok();
  ResolvedOpts r = loop ? loop->opts : resolve_opts(opts, dtype, STENCIL_OP_STEP, domain);
  r.dev = dev;
  // only the two-ended step reads a coefficient from device memory, whatever column
  // store the tuning table holds (a one-lane entry's 256-column tile serves it too)
  if (dev) r.column_store = STENCIL_COLUMN_SPLIT;
  if (variant_opts(opts)) {
    if (r.impl == STENCIL_IMPL_PLAIN)
      return fail(STENCIL_E_UNSUPPORTED, "the generalised diffusion runs the fused kernels only");
    if (domain[2] > split_step_limit((int)es))
      return fail(STENCIL_E_UNSUPPORTED, "the generalised step takes nk <= %d (nk = %lld)",
                  split_step_limit((int)es), (long long)domain[2]);
  }
  TRY(fused_nk_ok(r, domain));
  if (tile_narrow(r.tile_i, r.tile_j) && !narrow_tile_runs(r, STENCIL_OP_STEP, dtype, domain))
    return fail(STENCIL_E_UNSUPPORTED,
                "the %dx%d tile (128 columns) runs the fused two-ended step only (column store SPLIT, nk <= %d)",
                r.tile_i, r.tile_j, split_step_limit((int)es));
  if (r.impl == STENCIL_IMPL_PLAIN) TRY(need_plain_ws(r, plain_ws_bytes(es, domain)));
  TRY(check_device());
  r.wrapped = wrapped;
  TRY(dtype == STENCIL_F64 ? run_step<double>(u, data, w, out, domain, coeff, dt_dz, mask, r, stream)
                           : run_step<float>(u, data, w, out, domain, coeff, dt_dz, mask, r, stream));
  return periodic && !(loop && loop->wraps) ? stencil_halo_update(dtype, out, domain, STENCIL_BOUNDARY_PERIODIC, stream) : ok();
}

int stencil_step(stencil_dtype dtype, const stencil_field* u, const stencil_field* data,
                 const stencil_field* w, stencil_field* out, const int64_t domain[3], double coeff,
                 double dt_dz, void* mask, const stencil_options* opts, hipStream_t stream) {
  return step_call(dtype, u, data, w, out, domain, coeff, dt_dz, mask, opts, stream, nullptr);
}

}  // extern "C"

namespace gt4mi {

int plan_loop(stencil_dtype dtype, const int64_t* dom, const stencil_options* opts, LoopPlan* p) {
  TRY(check_opts(opts));
  p->opts = resolve_opts(opts, dtype, STENCIL_OP_STEP, dom);
  const ResolvedOpts& r = p->opts;
  // the two-ended step, and a period no shorter than the halo
  p->wraps = opts && opts->boundary == STENCIL_BOUNDARY_PERIODIC && !domain_empty(dom) &&
             r.impl != STENCIL_IMPL_PLAIN && (variant_opts(opts) || r.column_store == STENCIL_COLUMN_SPLIT) &&
             dom[2] <= split_step_limit((int)esize(dtype)) && dom[0] >= kHalo && dom[1] >= kHalo;
  return STENCIL_OK;
}

int loop_step(stencil_dtype dtype, const stencil_field* u, const stencil_field* data, const stencil_field* w,
              stencil_field* out, const int64_t* dom, double coeff, double dt_dz, const stencil_options* opts,
              const LoopPlan& p, bool first, hipStream_t stream) {
  return step_call(dtype, u, data, w, out, dom, coeff, dt_dz, nullptr, opts, stream, nullptr, &p, p.wraps && !first);
}

}  // namespace gt4mi

extern "C" {

int stencil_halo_update(stencil_dtype dtype, stencil_field* f, const int64_t domain[3], int boundary,
                        hipStream_t stream) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  if (boundary != STENCIL_BOUNDARY_FROZEN && boundary != STENCIL_BOUNDARY_PERIODIC)
    return fail(STENCIL_E_ARG, "boundary = %d unknown", boundary);
  TRY(check_field("f", f, domain, ROLE_HALO, esize(dtype)));
  if (boundary == STENCIL_BOUNDARY_FROZEN || domain_empty(domain)) return ok();
  TRY(check_device());
  const int ni = (int)domain[0], nj = (int)domain[1], nk = (int)domain[2];
  hipError_t e = dtype == STENCIL_F64
                     ? launch_halo_periodic<double>(at_origin_mut<double>(f), f->stride[1], f->stride[2], ni, nj, nk, stream)
                     : launch_halo_periodic<float>(at_origin_mut<float>(f), f->stride[1], f->stride[2], ni, nj, nk, stream);
  return hip_status(e, "periodic halo update");
}

static int hdiff_adjoint_call(stencil_dtype dtype, const stencil_field* out_bar, const void* mask,
                          stencil_field* u_bar, const int64_t domain[3], double coeff,
                          const stencil_options* opts, hipStream_t stream,
                  const DevCoeff* dev) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  TRY(check_opts(opts));
  const size_t es = esize(dtype);
  TRY(check_field("out_bar", out_bar, domain, ROLE_INTERIOR, es));
  TRY(check_field("u_bar", u_bar, domain, ROLE_HALO, es));
  const Span sb = span_of(u_bar, es);
  TRY(check_no_alias("u_bar", sb, "out_bar", span_of(out_bar, es)));
  TRY(check_coeff_field(opts, domain, es, "u_bar", sb));
  if (domain[2] == 0) return ok();
  const bool empty = domain_empty(domain);
  if (!mask && !empty) return fail(STENCIL_E_NULL, "mask is NULL");
  if (mask) {
    Span m{reinterpret_cast<uintptr_t>(mask), reinterpret_cast<uintptr_t>(mask) + stencil_mask_bytes(domain)};
    TRY(check_no_alias("u_bar", sb, "mask", m));
  }
  ResolvedOpts r = resolve_opts(opts, dtype, STENCIL_OP_HDIFF_ADJOINT, domain);
  r.dev = dev;
  TRY(check_device());
  if (dtype == STENCIL_F64) {
    return run_hdiff_adjoint<double>(at_origin<double>(out_bar), out_bar->stride[1], out_bar->stride[2],
                                     mask, u_bar, domain, coeff, r, stream);
  }
  return run_hdiff_adjoint<float>(at_origin<float>(out_bar), out_bar->stride[1], out_bar->stride[2],
                                  mask, u_bar, domain, coeff, r, stream);
}

int stencil_hdiff_adjoint(stencil_dtype dtype, const stencil_field* out_bar, const void* mask,
                          stencil_field* u_bar, const int64_t domain[3], double coeff,
                          const stencil_options* opts, hipStream_t stream) {
  return hdiff_adjoint_call(dtype, out_bar, mask, u_bar, domain, coeff, opts, stream, nullptr);
}

int stencil_vadv_adjoint(stencil_dtype dtype, const stencil_field* x_bar, const stencil_field* w,
                         stencil_field* d_bar, const int64_t domain[3], double dt_dz,
                         const stencil_options* opts, hipStream_t stream) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  TRY(check_opts(opts));
  const size_t es = esize(dtype);
  TRY(check_field("x_bar", x_bar, domain, ROLE_INTERIOR, es));
  TRY(check_field("w", w, domain, ROLE_STAGGERED, es));
  TRY(check_field("d_bar", d_bar, domain, ROLE_INTERIOR, es));
  const Span sd = span_of(d_bar, es);
  TRY(check_no_alias("d_bar", sd, "x_bar", span_of(x_bar, es)));
  TRY(check_no_alias("d_bar", sd, "w", span_of(w, es)));
  if (domain_empty(domain)) return ok();
  ResolvedOpts r = resolve_opts(opts, dtype, STENCIL_OP_VADV_ADJOINT, domain);
  const bool plain = r.impl == STENCIL_IMPL_PLAIN || domain[2] > kMaxFusedNk;
  if (r.impl == STENCIL_IMPL_FUSED && domain[2] > kMaxFusedNk)
    return fail(STENCIL_E_UNSUPPORTED, "nk = %lld exceeds the fused column limit %d", (long long)domain[2], kMaxFusedNk);
  TRY(need_plain_ws(r, adj_ws_bytes(es, domain, false, plain)));
  TRY(check_device());
  if (dtype == STENCIL_F64)
    return run_vadv_adjoint<double>(x_bar, w, at_origin_mut<double>(d_bar), d_bar->stride[1], d_bar->stride[2],
                                    domain, dt_dz, r, r.ws, stream);
  return run_vadv_adjoint<float>(x_bar, w, at_origin_mut<float>(d_bar), d_bar->stride[1], d_bar->stride[2],
                                 domain, dt_dz, r, r.ws, stream);
}

static int step_adjoint_call(stencil_dtype dtype, const stencil_field* x_bar, const stencil_field* w,
                         const void* mask, stencil_field* u_bar, stencil_field* data_bar,
                         const int64_t domain[3], double coeff, double dt_dz,
                         const stencil_options* opts, hipStream_t stream,
                  const DevCoeff* dev) {
  TRY(check_dtype(dtype));
  TRY(check_domain(domain));
  TRY(check_opts(opts));
  const size_t es = esize(dtype);
  TRY(check_field("x_bar", x_bar, domain, ROLE_INTERIOR, es));
  TRY(check_field("w", w, domain, ROLE_STAGGERED, es));
  TRY(check_field("u_bar", u_bar, domain, ROLE_HALO, es));
  const Span sb = span_of(u_bar, es), sx = span_of(x_bar, es), sw = span_of(w, es);
  TRY(check_no_alias("u_bar", sb, "x_bar", sx));
  TRY(check_no_alias("u_bar", sb, "w", sw));
  if (data_bar) {
    TRY(check_field("data_bar", data_bar, domain, ROLE_INTERIOR, es));
    const Span sd = span_of(data_bar, es);
    TRY(check_no_alias("data_bar", sd, "x_bar", sx));
    TRY(check_no_alias("data_bar", sd, "w", sw));
    TRY(check_no_alias("data_bar", sd, "u_bar", sb));
    TRY(check_coeff_field(opts, domain, es, "data_bar", sd));
  }
  TRY(check_coeff_field(opts, domain, es, "u_bar", sb));
  if (domain[2] == 0) return ok();
  const bool empty = domain_empty(domain);
  if (!mask && !empty) return fail(STENCIL_E_NULL, "mask is NULL");
  if (mask) {
    Span m{reinterpret_cast<uintptr_t>(mask), reinterpret_cast<uintptr_t>(mask) + stencil_mask_bytes(domain)};
    TRY(check_no_alias("u_bar", sb, "mask", m));
  }
  ResolvedOpts r = resolve_opts(opts, dtype, STENCIL_OP_STEP_ADJOINT, domain);
  r.dev = dev;
  const bool plain = r.impl == STENCIL_IMPL_PLAIN || domain[2] > kMaxFusedNk;
  if (r.impl == STENCIL_IMPL_FUSED && domain[2] > kMaxFusedNk)
    return fail(STENCIL_E_UNSUPPORTED, "nk = %lld exceeds the fused column limit %d", (long long)domain[2], kMaxFusedNk);
  const size_t need = adj_ws_bytes(es, domain, data_bar == nullptr, plain);
  TRY(need_plain_ws(r, need));
  if (r.ws && need) {
    Span swsp{reinterpret_cast<uintptr_t>(r.ws), reinterpret_cast<uintptr_t>(r.ws) + need};
    TRY(check_no_alias("workspace", swsp, "u_bar", sb));
    TRY(check_no_alias("workspace", swsp, "x_bar", sx));
    TRY(check_no_alias("workspace", swsp, "w", sw));
  }
  TRY(check_device());
  const int64_t n = domain[0] * domain[1] * domain[2];
  auto go = [&](auto tag) -> int {
    using T = decltype(tag);
    T* lam;
    int64_t l_sj, l_sk;
    char* rest = static_cast<char*>(r.ws);
    if (data_bar) {
      lam = at_origin_mut<T>(data_bar);
      l_sj = data_bar->stride[1];
      l_sk = data_bar->stride[2];
    } else if (empty) {
      lam = nullptr;  // no interior: the gather reads no lambda, it only zeroes u_bar
      l_sj = l_sk = 0;
    } else {
      lam = static_cast<T*>(r.ws);
      l_sj = domain[0];
      l_sk = domain[0] * domain[1];
      rest += r256(n * (int64_t)sizeof(T));
    }
    if (!empty) TRY(run_vadv_adjoint<T>(x_bar, w, lam, l_sj, l_sk, domain, dt_dz, r, rest, stream));
    return run_hdiff_adjoint<T>(lam, l_sj, l_sk, mask, u_bar, domain, coeff, r, stream);
  };
  return dtype == STENCIL_F64 ? go(double(0)) : go(float(0));
}

int stencil_step_adjoint(stencil_dtype dtype, const stencil_field* x_bar, const stencil_field* w,
                         const void* mask, stencil_field* u_bar, stencil_field* data_bar,
                         const int64_t domain[3], double coeff, double dt_dz,
                         const stencil_options* opts, hipStream_t stream) {
  return step_adjoint_call(dtype, x_bar, w, mask, u_bar, data_bar, domain, coeff, dt_dz, opts, stream, nullptr);
}

// ------------------------------------------------------------------ training calls
// Fields over contiguous (k, j, i) buffers: h points of halo, `extra` more levels.
static stencil_field dense(const void* p, const int64_t* dom, int h, int extra) {
  const int64_t x = dom[0] + 2 * h, y = dom[1] + 2 * h;
  return stencil_field{const_cast<void*>(p), {x, y, dom[2] + extra}, {1, x, x * y}, {h, h, 0}};
}

// The buffers of one call that are there, for the check that no output overlaps
// an input or another output.
namespace {
struct Buffers {
  struct { const char* name; Span s; } v[8];
  int n = 0;
  void add(const char* name, const void* p, size_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    if (p && bytes) v[n].name = name, v[n++].s = Span{a, a + bytes};
  }
  void add(const char* name, const stencil_field& f, size_t es) {
    if (f.data) v[n].name = name, v[n++].s = span_of(&f, es);
  }
};

int check_outputs(const Buffers& out, const Buffers& in) {
  for (int o = 0; o < out.n; ++o) {
    for (int i = 0; i < in.n; ++i) TRY(check_no_alias(out.v[o].name, out.v[o].s, in.v[i].name, in.v[i].s));
    for (int q = o + 1; q < out.n; ++q) TRY(check_no_alias(out.v[o].name, out.v[o].s, out.v[q].name, out.v[q].s));
  }
  return STENCIL_OK;
}

int check_aligned(const char* name, const void* p, size_t bytes) {
  if (reinterpret_cast<uintptr_t>(p) % bytes)
    return fail(STENCIL_E_DTYPE, "%s is not aligned to %zu bytes", name, bytes);
  return STENCIL_OK;
}
}  // namespace

int stencil_train_forward(stencil_dtype dtype, const void* u, const void* data, const void* w, void* out,
                          void* mask, const void* kappa, double coeff, const void* coeff_dev,
                          stencil_dtype coeff_dtype, void* coeff_copy, int64_t ni, int64_t nj, int64_t nk,
                          double dt_dz, int form, hipStream_t stream) {
  const int64_t dom[3] = {ni, nj, nk};
  TRY(check_dtype(dtype));
  TRY(check_domain(dom));
  if (coeff_dev) {
    if (kappa) return fail(STENCIL_E_ARG, "both a coefficient field and a scalar coefficient in device memory");
    TRY(check_dtype(coeff_dtype));
    if (!mask) return fail(STENCIL_E_NULL, "mask is NULL");
    if (!coeff_copy) return fail(STENCIL_E_NULL, "coeff_copy is NULL");
    if (w && nk > split_step_limit((int)esize(dtype)))
      return fail(STENCIL_E_UNSUPPORTED, "a coefficient in device memory takes nk <= %d", split_step_limit((int)esize(dtype)));
  }
  const stencil_field fu = dense(u, dom, 2, 0), fk = dense(kappa, dom, 0, 0);
  const stencil_field fd = dense(data, dom, 0, 0), fw = dense(w, dom, 0, 1);
  stencil_field fo = dense(out, dom, 0, 0);
  if (coeff_dev) {
    const size_t es = esize(dtype), cs = esize(coeff_dtype);
    TRY(check_aligned("coeff_dev", coeff_dev, cs));
    TRY(check_aligned("coeff_copy", coeff_copy, es));
    TRY(check_field("u", &fu, dom, ROLE_HALO, es));
    TRY(check_field("out", &fo, dom, ROLE_INTERIOR, es));
    if (w) {
      TRY(check_field("data", &fd, dom, ROLE_INTERIOR, es));
      TRY(check_field("w", &fw, dom, ROLE_STAGGERED, es));
    }
    Buffers in, outs;
    in.add("coeff_dev", coeff_dev, cs);
    in.add("u", fu, es);
    if (w) in.add("data", fd, es);
    if (w) in.add("w", fw, es);
    outs.add("coeff_copy", coeff_copy, es);
    outs.add("out", fo, es);
    outs.add("mask", mask, stencil_mask_bytes(dom));
    if (!domain_empty(dom)) TRY(check_outputs(outs, in));
  }
  stencil_options o;
  memset(&o, 0, sizeof o);
  o.hdiff_form = form;
  o.coeff_field = kappa ? const_cast<stencil_field*>(&fk) : nullptr;
  const DevCoeff dev{coeff_dev, coeff_dtype == STENCIL_F64, coeff_copy};
  const DevCoeff* d = coeff_dev ? &dev : nullptr;
  if (!w) return hdiff_call(dtype, &fu, &fo, dom, coeff, mask, &o, stream, d);
  return step_call(dtype, &fu, &fd, &fw, &fo, dom, coeff, dt_dz, mask, &o, stream, d);
}

int stencil_train_backward(stencil_dtype dtype, const void* x_bar, const void* mask, const void* u, const void* w,
                           const void* x, const void* kappa, double coeff, const void* coeff_copy, void* u_bar,
                           void* data_bar, void* w_bar, void* kappa_bar, void* coeff_bar, void* ws,
                           size_t ws_bytes, int64_t ni, int64_t nj, int64_t nk, double dt_dz, int form,
                           hipStream_t stream) {
  const int64_t dom[3] = {ni, nj, nk};
  TRY(check_dtype(dtype));
  TRY(check_domain(dom));
  if ((kappa_bar || coeff_bar) && !u) return fail(STENCIL_E_NULL, "u is NULL");
  if (w_bar && !(w && x)) return fail(STENCIL_E_NULL, "w_bar needs w and x");
  if (coeff_bar && kappa) return fail(STENCIL_E_ARG, "a coefficient field has no scalar coeff_bar");
  if (coeff_copy && kappa) return fail(STENCIL_E_ARG, "both a coefficient field and a scalar coefficient in device memory");
  const size_t es = esize(dtype), need = coeff_bar ? stencil_param_workspace_bytes(dtype, dom) : 0;
  if (need) {
    if (!ws) return fail(STENCIL_E_WORKSPACE, "coeff_bar needs %zu bytes of workspace (ws is NULL)", need);
    if (ws_bytes < need)
      return fail(STENCIL_E_WORKSPACE, "workspace of %zu bytes is smaller than the %zu needed", ws_bytes, need);
    if (reinterpret_cast<uintptr_t>(ws) % 8) return fail(STENCIL_E_WORKSPACE, "workspace is not 8-byte aligned");
  }
  TRY(check_aligned("coeff_copy", coeff_copy, es));
  TRY(check_aligned("coeff_bar", coeff_bar, es));
  const stencil_field fx = dense(x_bar, dom, 0, 0), fk = dense(kappa, dom, 0, 0), fw = dense(w, dom, 0, 1);
  const stencil_field fu = dense(u, dom, 2, 0), fo = dense(x, dom, 0, 0);
  stencil_field fb = dense(u_bar, dom, 2, 0), fd = dense(data_bar, dom, 0, 0);
  stencil_field kb = dense(kappa_bar, dom, 0, 0), wb = dense(w_bar, dom, 0, 1);
  {
    Buffers in, out;
    auto field = [&](Buffers& set, const char* name, const stencil_field& f, Role role) -> int {
      TRY(check_field(name, &f, dom, role, es));
      set.add(name, f, es);
      return STENCIL_OK;
    };
    TRY(field(in, "x_bar", fx, ROLE_INTERIOR));
    TRY(field(out, "u_bar", fb, ROLE_HALO));
    if (w) TRY(field(in, "w", fw, ROLE_STAGGERED));
    if (w) TRY(field(out, "data_bar", fd, ROLE_INTERIOR));
    if (kappa) TRY(field(in, "kappa", fk, ROLE_INTERIOR));
    if (kappa_bar || coeff_bar) TRY(field(in, "u", fu, ROLE_HALO));
    if (w_bar) TRY(field(in, "x", fo, ROLE_INTERIOR));
    if (w_bar) TRY(field(out, "w_bar", wb, ROLE_STAGGERED));
    if (kappa_bar) TRY(field(out, "kappa_bar", kb, ROLE_INTERIOR));
    in.add("mask", mask, stencil_mask_bytes(dom));
    in.add("coeff_copy", coeff_copy, es);
    out.add("coeff_bar", coeff_bar, es);
    out.add("the workspace", ws, need);
    if (!domain_empty(dom)) TRY(check_outputs(out, in));
  }
  stencil_options o;
  memset(&o, 0, sizeof o);
  o.hdiff_form = form;
  o.coeff_field = kappa ? const_cast<stencil_field*>(&fk) : nullptr;
  const DevCoeff dev{coeff_copy, false, nullptr};
  const DevCoeff* d = coeff_copy ? &dev : nullptr;
  if (w) TRY(step_adjoint_call(dtype, &fx, &fw, mask, &fb, &fd, dom, coeff, dt_dz, &o, stream, d));
  else TRY(hdiff_adjoint_call(dtype, &fx, mask, &fb, dom, coeff, &o, stream, d));
  if (!kappa_bar && !coeff_bar && !w_bar) return ok();
  auto go = [&](auto tag) -> int {
    using T = decltype(tag);
    const stencil_field lam = w ? fd : fx;
    StepArgs<T> A = step_args<T>(u ? &fu : nullptr, &lam, nullptr, kappa_bar ? &kb : nullptr, dom, 0.0, dt_dz, nullptr);
    A.form = form;
    if (kappa_bar && !domain_empty(dom)) TRY(hip_status(launch_coeff_field_grad<T>(A, stream), "coefficient field gradient"));
    if (!coeff_bar && !w_bar) return ok();
    WGradArgs<T> W;
    if (w_bar) W = w_grad_args<T>(&fw, &fo, &lam, &wb, dom, dt_dz);
    return hip_status(launch_param_grads<T>(A, w_bar ? &W : nullptr, static_cast<double*>(ws), (int64_t)(need / 8),
                                            coeff_bar, dtype == STENCIL_F32, stream),
                      "step parameter gradients");
  };
  return dtype == STENCIL_F64 ? go(double(0)) : go(float(0));
}

}  // extern "C"
