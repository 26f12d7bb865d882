// capi.cpp -- C-ABI of libgsis.so: argument checks, plan set-up (ordinate
// regrouping, least-squares / synthetic coefficients, multigrid hierarchy)
// and the outer-iteration driver. Every arithmetic step of an iteration runs
// in the HIP kernels; the host only sets up coefficients once per plan.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/gsis.h"
#include "plan.h"

thread_local std::string g_create_err;

extern "C" {

const char *gsis_version(void) {
  return "libgsis (HIP, gfx950) FP64 wavefront sweep + CG/GMG synthetic solve";
}

gsis_status gsis_ctx_create(int32_t device, gsis_ctx **out) {
  if (!out) return fail(nullptr, GSIS_E_INVALID_ARG, "out is NULL");
  int n = 0;
  hipError_t e = hipGetDeviceCount(&n);
  if (e != hipSuccess || n == 0)
    return fail(nullptr, GSIS_E_DEVICE, "no HIP device: %s", hipGetErrorString(e));
  if (device < 0 || device >= n)
    return fail(nullptr, GSIS_E_INVALID_ARG, "device %d out of range [0,%d)", device, n);
  e = hipSetDevice(device);
  if (e != hipSuccess) return fail(nullptr, GSIS_E_DEVICE, "hipSetDevice: %s", hipGetErrorString(e));
  gsis_ctx *c = new gsis_ctx;
  c->device = device;
  *out = c;
  return GSIS_OK;
}

void gsis_ctx_destroy(gsis_ctx *ctx) { delete ctx; }

const char *gsis_last_error(const gsis_ctx *ctx) {
  return ctx ? ctx->err.c_str() : g_create_err.c_str();
}

gsis_status gsis_options_default(gsis_options *o) {
  if (!o) return GSIS_E_INVALID_ARG;
  std::memset(o, 0, sizeof *o);
  o->method = GSIS_GSIS;
  o->precision = GSIS_FP64;
  o->order = 2;
  o->limiter = 1;
  o->alsm = 1;
  o->hot_face = GSIS_HOT_CENTRAL;
  o->tol = 1e-6;
  o->max_iter = 1000;
  o->synth_rtol = 0.1;
  o->synth_max_iter = 50;
  o->cfl_p = 0.0;
  o->beta = 0.0;
  o->graph = 1;
  o->synth_form = 0;
  o->synth_sub = 4;
  return GSIS_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ helpers
namespace {

// Copy n doubles from caller memory (host or device) to a host vector.
gsis_status fetch(gsis_ctx *ctx, const double *src, size_t n, int dev, std::vector<double> &dst,
                  const char *name) {
  if (!src) return fail(ctx, GSIS_E_INVALID_ARG, "%s is NULL", name);
  dst.resize(n);
  if (n == 0) return GSIS_OK;
  if (dev) {
    hipError_t e = hipMemcpy(dst.data(), src, n * sizeof(double), hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
      (void)hipGetLastError();   // (not for the next call to find)
      return fail(ctx, GSIS_E_DEVICE, "reading %s: %s", name, hipGetErrorString(e));
    }
  } else {
    std::memcpy(dst.data(), src, n * sizeof(double));
  }
  return GSIS_OK;
}

// Everything about the problem but its cell and boundary fields, which
// plan_create checks (on the device where they are there, launch_check_cells and
// launch_setup_bnd).
gsis_status check_problem(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                          std::vector<double> &mu, std::vector<double> &eta,
                          std::vector<double> &w) {
  if (!p) return fail(ctx, GSIS_E_INVALID_ARG, "problem is NULL");
  if (!o) return fail(ctx, GSIS_E_INVALID_ARG, "options is NULL");
  if (p->nx < 1 || p->ny < 1)
    return fail(ctx, GSIS_E_INVALID_ARG, "nx, ny must be >= 1 (got %d, %d)", p->nx, p->ny);
  if ((long long)p->nx * p->ny > GSIS_MAX_CELLS)
    return fail(ctx, GSIS_E_INVALID_ARG, "nx*ny = %lld too large (at most %d cells)",
                (long long)p->nx * p->ny, GSIS_MAX_CELLS);
  if (!(p->dx > 0) || !(p->dy > 0) || !std::isfinite(p->dx) || !std::isfinite(p->dy))
    return fail(ctx, GSIS_E_INVALID_ARG, "dx, dy must be finite and > 0");
  if (p->K < 1) return fail(ctx, GSIS_E_INVALID_ARG, "K must be >= 1 (got %d)", p->K);
  if (o->method != GSIS_SI && o->method != GSIS_GSIS)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.method must be 0 or 1");
  if (o->precision != GSIS_FP64 && o->precision != GSIS_FP32_MIXED)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.precision must be 0 or 1");
  if (o->order != 1 && o->order != 2)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.order must be 1 or 2");
  if (o->hot_face != GSIS_HOT_CENTRAL && o->hot_face != GSIS_HOT_TRANSPORT)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.hot_face must be 0 or 1");
  if (o->max_iter < 1) return fail(ctx, GSIS_E_INVALID_ARG, "options.max_iter must be >= 1");
  if (!(o->tol >= 0) || std::isnan(o->tol))
    return fail(ctx, GSIS_E_INVALID_ARG, "options.tol must be >= 0");
  if (!(o->synth_rtol > 0)) return fail(ctx, GSIS_E_INVALID_ARG, "options.synth_rtol must be > 0");
  if (o->synth_max_iter < 1)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.synth_max_iter must be >= 1");
  if (!(o->cfl_p >= 0) || !std::isfinite(o->cfl_p))
    return fail(ctx, GSIS_E_INVALID_ARG, "options.cfl_p must be finite and >= 0");
  if (!(o->beta >= 0) || !std::isfinite(o->beta))
    return fail(ctx, GSIS_E_INVALID_ARG, "options.beta must be finite and >= 0");
  if (o->synth_form != 0 && o->synth_form != 1)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.synth_form must be 0 or 1");
  if (o->synth_form == 1 && o->synth_sub < 1)
    return fail(ctx, GSIS_E_INVALID_ARG, "options.synth_sub must be >= 1");
  const int dev = o->device_ptrs;
  const size_t K = p->K;
  gsis_status st;
  if ((st = fetch(ctx, p->mu, K, dev, mu, "mu")) || (st = fetch(ctx, p->eta, K, dev, eta, "eta")) ||
      (st = fetch(ctx, p->w, K, dev, w, "w")))
    return st;
  if (!p->sigma_a) return fail(ctx, GSIS_E_INVALID_ARG, "sigma_a is NULL");
  if (!p->sigma_s) return fail(ctx, GSIS_E_INVALID_ARG, "sigma_s is NULL");
  if (!p->q) return fail(ctx, GSIS_E_INVALID_ARG, "q is NULL");
  double wsum = 0;
  for (size_t k = 0; k < K; ++k) {
    if (!std::isfinite(mu[k]) || !std::isfinite(eta[k]) || !std::isfinite(w[k]))
      return fail(ctx, GSIS_E_INVALID_ARG, "quadrature entry %zu is not finite", k);
    if (mu[k] * mu[k] + eta[k] * eta[k] > 1.0 + 1e-12)
      return fail(ctx, GSIS_E_INVALID_ARG, "mu[%zu]^2 + eta[%zu]^2 > 1", k, k);
    if (w[k] < 0) return fail(ctx, GSIS_E_INVALID_ARG, "w[%zu] < 0", k);
    wsum += w[k];
  }
  if (std::fabs(wsum - kFourPi) > 1e-12 * kFourPi)
    return fail(ctx, GSIS_E_INVALID_ARG, "sum(w) = %.17g, expected 4*pi", wsum);
  return GSIS_OK;
}

// A kernel on the context's device can read and write p: memory of that
// device, or host memory that is mapped for it. Memory of another device or
// pageable host memory passed with device_ptrs is left to the runtime's copies,
// which take it or return an error.
bool kernel_reaches(const gsis_ctx *ctx, const void *p) {
  if (!p) return true;
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (a.type == hipMemoryTypeManaged) return true;
  if (a.type == hipMemoryTypeHost) return a.devicePointer == p;
  return a.type == hipMemoryTypeDevice && a.device == ctx->device;
}

// Copies n doubles of the caller (host or device) to the device on s.
gsis_status fetch_dev(gsis_plan *pl, const double *src, double *dst, size_t n, const char *name) {
  if (pl->device_ptrs && !kernel_reaches(pl->ctx, src)) {
    std::vector<double> h;
    gsis_status st = fetch(pl->ctx, src, n, 1, h, name);
    if (st) return st;
    HIPCHK(pl->ctx, hipMemcpy(dst, h.data(), n * sizeof(double), hipMemcpyHostToDevice));
    return GSIS_OK;
  }
  const hipError_t e =
      hipMemcpyAsync(dst, src, n * sizeof(double),
                     pl->device_ptrs ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, pl->stream);
  if (e != hipSuccess)
    return fail(pl->ctx, GSIS_E_DEVICE, "reading %s: %s", name, hipGetErrorString(e));
  return GSIS_OK;
}

// One intensity buffer: N*K doubles, or N*K floats in FP32-mixed mode.
gsis_status alloc_intensity(gsis_plan *pl, int which, size_t nk, bool f32) {
  gsis_status st;
  if (f32) {
    float *p = nullptr;
    st = dalloc(pl, &p, nk);
    pl->P.I[which] = p;
  } else {
    double *p = nullptr;
    st = dalloc(pl, &p, nk);
    pl->P.I[which] = p;
  }
  return st;
}

// Dense SPD inverse by Cholesky (coarsest multigrid level, n <= a few hundred).
bool dense_spd_inverse(int n, std::vector<double> &A) {
  std::vector<double> L(A);
  for (int j = 0; j < n; ++j) {
    double s = L[(size_t)j * n + j];
    for (int k = 0; k < j; ++k) s -= L[(size_t)j * n + k] * L[(size_t)j * n + k];
    if (!(s > 0)) return false;
    const double d = std::sqrt(s);
    L[(size_t)j * n + j] = d;
    for (int i = j + 1; i < n; ++i) {
      double t = L[(size_t)i * n + j];
      for (int k = 0; k < j; ++k) t -= L[(size_t)i * n + k] * L[(size_t)j * n + k];
      L[(size_t)i * n + j] = t / d;
    }
  }
  // A^{-1}: solve L L^T X = 1, all columns side by side
  for (int i = 0; i < n; ++i) {
    double *x = &A[(size_t)i * n];
    for (int c = 0; c < n; ++c) x[c] = i == c ? 1.0 : 0.0;
    for (int k = 0; k < i; ++k) {
      const double l = L[(size_t)i * n + k], *y = &A[(size_t)k * n];
      for (int c = 0; c < n; ++c) x[c] -= l * y[c];
    }
    const double d = L[(size_t)i * n + i];
    for (int c = 0; c < n; ++c) x[c] /= d;
  }
  for (int i = n - 1; i >= 0; --i) {
    double *x = &A[(size_t)i * n];
    for (int k = i + 1; k < n; ++k) {
      const double l = L[(size_t)k * n + i], *y = &A[(size_t)k * n];
      for (int c = 0; c < n; ++c) x[c] -= l * y[c];
    }
    const double d = L[(size_t)i * n + i];
    for (int c = 0; c < n; ++c) x[c] /= d;
  }
  return true;
}


}  // namespace

namespace {

gsis_status alloc_level(gsis_plan *pl, MGLevel &L) {
  const size_t n = (size_t)L.nx * L.ny;
  gsis_status st;
  if ((st = dalloc(pl, &L.diag, 3 * n))) return st;   // the operator in one piece
  L.ax = L.diag + op_ax((int)n);
  L.ay = L.diag + op_ay((int)n);
  if ((st = dalloc(pl, &L.x, n)) || (st = dalloc(pl, &L.b, n)) || (st = dalloc(pl, &L.r, n)))
    return st;
  return GSIS_OK;
}

// Aggregates of level F: 2x2, or 2x1 / 1x2 when the couplings in one
// direction are much weaker than in the other (then merging across the weak
// direction would leave error the point smoother cannot reach), by the
// geometric means of the couplings. The device's sums of logarithms decide
// unless they are so close to the threshold that their rounding could; then
// the sums are formed on the host, cell by cell (a uniform medium on cells of
// aspect ratio 2 sits on the threshold).
gsis_status choose_aggregates(gsis_plan *pl, MGLevel &F, double *part) {
  gsis_ctx *ctx = pl->ctx;
  const long mx = (long)(F.nx - 1) * F.ny, my = (long)F.nx * (F.ny - 1);
  const int nb = launch_log_sums(F, part, pl->stream);
  std::vector<double> h(2 * (size_t)nb);
  HIPCHK(ctx, hipMemcpyAsync(h.data(), part, h.size() * sizeof(double), hipMemcpyDeviceToHost,
                             pl->stream));
  HIPCHK(ctx, hipStreamSynchronize(pl->stream));
  double lx = 0, ly = 0;
  for (int b = 0; b < nb; ++b) { lx += h[2 * b]; ly += h[2 * b + 1]; }
  if (mx && my) {
    const double r = lx / mx - ly / my, thr = std::log(0.25);
    if (!(std::fabs(r - thr) > 1e-9 && std::fabs(-r - thr) > 1e-9)) {
      const size_t n = (size_t)F.nx * F.ny;
      std::vector<double> a(2 * n);
      static_assert(op_ax(1) == op_ay(1) + 1, "ax behind ay");
      HIPCHK(ctx, hipMemcpyAsync(a.data(), F.ay, 2 * n * sizeof(double), hipMemcpyDeviceToHost,
                                 pl->stream));
      HIPCHK(ctx, hipStreamSynchronize(pl->stream));
      lx = ly = 0;
      for (int j = 0; j < F.ny; ++j)
        for (int i = 0; i < F.nx; ++i) {
          const size_t c = (size_t)j * F.nx + i;
          if (i + 1 < F.nx) lx += std::log(a[n + c]);
          if (j + 1 < F.ny) ly += std::log(a[c]);
        }
    }
  }
  const double gx = mx ? std::exp(lx / mx) : 0.0, gy = my ? std::exp(ly / my) : 0.0;
  F.fx = (F.nx > 1 && gx >= 0.25 * gy) ? 2 : 1;
  F.fy = (F.ny > 1 && gy >= 0.25 * gx) ? 2 : 1;
  return GSIS_OK;
}

// Multigrid hierarchy of the level-0 synthetic operator P.mg[0] (Galerkin
// coarsening) and the device state of a synthetic solve on P: levels, dense
// coarsest inverse, CG vectors, block partials and scalars. P.N must be set.
gsis_status setup_synth(gsis_plan *pl, PlanDev &P) {
  gsis_ctx *ctx = pl->ctx;
  gsis_status st;
  const int kCoarseMax = 64;   // dense inverse of the coarsest level: at most 64 x 64
  double *part = P.mom_part;   // (12 N values, not in use yet)
  static_assert(12 * kCoarseMax >= 2 * kLogBlocks, "partial sums of a level above the coarsest");
  while ((long)P.mg.back().nx * P.mg.back().ny > kCoarseMax &&
         (P.mg.back().nx > 1 || P.mg.back().ny > 1)) {
    if ((st = choose_aggregates(pl, P.mg.back(), part))) return st;
    const MGLevel F = P.mg.back();
    MGLevel C;
    C.nx = (F.nx + F.fx - 1) / F.fx;
    C.ny = (F.ny + F.fy - 1) / F.fy;
    if ((st = alloc_level(pl, C))) return st;
    launch_coarsen(F, C, pl->stream);
    P.mg.push_back(C);
    if (P.mg.size() > (size_t)kMaxLevels)
      return fail(ctx, GSIS_E_INVALID_ARG, "multigrid hierarchy deeper than %d levels", kMaxLevels);
  }
  // dense inverse of the coarsest level
  const MGLevel &Lc = P.mg.back();
  const int nc = Lc.nx * Lc.ny;
  std::vector<double> op(3 * (size_t)nc), dense((size_t)nc * nc, 0.0);
  HIPCHK(ctx, hipMemcpyAsync(op.data(), Lc.diag, op.size() * sizeof(double), hipMemcpyDeviceToHost,
                             pl->stream));
  HIPCHK(ctx, hipStreamSynchronize(pl->stream));
  for (int j = 0; j < Lc.ny; ++j)
    for (int i = 0; i < Lc.nx; ++i) {
      const int c = j * Lc.nx + i;
      dense[(size_t)c * nc + c] = op[c];
      if (i + 1 < Lc.nx) {
        dense[(size_t)c * nc + c + 1] = -op[op_ax(nc) + c];
        dense[(size_t)(c + 1) * nc + c] = -op[op_ax(nc) + c];
      }
      if (j + 1 < Lc.ny) {
        dense[(size_t)c * nc + c + Lc.nx] = -op[op_ay(nc) + c];
        dense[(size_t)(c + Lc.nx) * nc + c] = -op[op_ay(nc) + c];
      }
    }
  if (!dense_spd_inverse(nc, dense))
    return fail(ctx, GSIS_E_INVALID_ARG, "synthetic operator is not positive definite");

  const int N = P.N;
  if ((st = dalloc(pl, &P.cg_r, N)) || (st = dalloc(pl, &P.cg_r2, N)) ||
      (st = dalloc(pl, &P.cg_z, N)) ||
      (st = dalloc(pl, &P.cg_p, N)) || (st = dalloc(pl, &P.cg_s0, N)) ||
      (st = dalloc(pl, &P.cg_s1, N)) || (st = dalloc(pl, &P.cg_w, N)) ||
      (st = dalloc(pl, &P.scal, 16)))
    return st;
  if (P.synth_form == 1 &&
      ((st = dalloc(pl, &P.wide_wx, N)) || (st = dalloc(pl, &P.wide_wy, N))))
    return st;
  // block partials: r.r and b.b (one per 256 cells each), then r.z, the
  // r.r of the level-0 tile kernel and z.Az (one per level-0 multigrid tile
  // each)
  P.red_blocks = (N + 255) / 256;
  const size_t ntp = std::max<size_t>(tiles_of(P.nx, P.ny), P.red_blocks);
  if ((st = dalloc(pl, &P.red, 2 * (size_t)P.red_blocks + 3 * ntp + 2))) return st;
  P.coarse_n = nc;
  return upload(pl, &P.coarse_inv, dense);
}

}  // namespace

// Launch set of a single plan: its synthetic-step descriptor on the device
// and block counts per level (no block tables). Needs every array of P.
gsis_status make_single_set(gsis_plan *pl) {
  PlanDev &P = pl->P;
  SynthSet &S = P.S;
  const SynthDesc D = make_synth_desc(P);
  gsis_status st;
  {
    char *d = nullptr;
    if ((st = dalloc(pl, &d, sizeof D))) return st;
    HIPCHK(pl->ctx, hipMemcpy(d, &D, sizeof D, hipMemcpyHostToDevice));
    S.desc = (SynthDesc *)d;
  }
  auto nb = [](int n) { return (n + 255) / 256; };
  S.n = 1;
  S.max_lc = D.lc;
  S.min_lc = D.lc;
  S.any_coef_sep = D.coef_sep == kCoefKernel;
  S.any_zw = needs_zw(D);
  S.any_sums = D.coef_sep == kCoefCoarse;
  P.lc = D.lc;
  S.coarse_lds = coarse_lds_bytes(P);
  S.coarse_cells = coarse_cells(P);
  S.whole = P.precision == GSIS_FP64;
  S.synth_max_iter = P.synth_max_iter;
  S.nb_cell = nb(P.N);
  S.bt_cell = nullptr;
  S.nb_src = source_tiles_of(P.nx, P.ny);
  S.bt_src = nullptr;
  S.bt_tile.assign(D.lc, nullptr);
  S.nb_tile.resize(D.lc);
  for (int l = 0; l < D.lc; ++l) S.nb_tile[l] = tiles_of(P.mg[l].nx, P.mg[l].ny);
  S.state0 = P.state;
  prepare_synth(S.coarse_lds);
  return GSIS_OK;
}

// ------------------------------------------------------------------- plans
// room for the partial sums of w r^2 of either residual kernel (a batch
// runs its own on a plan made for the pipelined step)
static size_t tres_slots(const PlanDev &P) {
  return std::max((size_t)P.n_tres, (size_t)P.n_rtiles * residual_pairs(P));
}

// A plan whose device memory comes from hipMalloc (arena NULL) or is carved
// from the arena_cap bytes at arena (no device or pinned allocation at all;
// profiling off; no adjoint; reset once, here).
// With mt, the time-dependent form (backward-Euler steps of size mt->dt).
// share: plans that run together (a batch).
// lean: the same phi and F from less memory (one moment partial per quadrant,
// no shorter residual tiles than of 31 diagonals), for a region that the form
// that runs fastest does not fit. *full: an array did not fit the region.
static gsis_status plan_create(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                               gsis_plan **out, char *arena, size_t arena_cap,
                               const gsis_material *mt = nullptr, int share = 1,
                               bool lean = false, bool *full = nullptr) {
  if (!ctx) return fail(nullptr, GSIS_E_INVALID_ARG, "ctx is NULL");
  if (!out) return fail(ctx, GSIS_E_INVALID_ARG, "out is NULL");
  *out = nullptr;
  std::vector<double> mu, eta, w;
  gsis_status st = check_problem(ctx, p, o, mu, eta, w);
  if (st) return st;
  if (mt) {
    if (!(mt->c > 0) || !std::isfinite(mt->c))
      return fail(ctx, GSIS_E_INVALID_ARG, "material.c must be finite and > 0");
    if (!(mt->a >= 0) || !std::isfinite(mt->a))
      return fail(ctx, GSIS_E_INVALID_ARG, "material.a must be finite and >= 0");
    if (!(mt->dt > 0) || !std::isfinite(mt->dt) || !std::isfinite(1.0 / (mt->c * mt->dt)))
      return fail(ctx, GSIS_E_INVALID_ARG, "material.dt must be finite and > 0");
    if (mt->sub_iter < 1) return fail(ctx, GSIS_E_INVALID_ARG, "material.sub_iter must be >= 1");
    if (o->precision != GSIS_FP64)
      return fail(ctx, GSIS_E_UNSUPPORTED, "the time-dependent form runs in FP64 only");
    if (o->synth_form != 0)
      return fail(ctx, GSIS_E_UNSUPPORTED, "the time-dependent form needs options.synth_form 0");
    if (!mt->cv) return fail(ctx, GSIS_E_INVALID_ARG, "material.cv is NULL");
    if (!mt->T0) return fail(ctx, GSIS_E_INVALID_ARG, "material.T0 is NULL");
  }
  if (o->method == GSIS_GSIS && o->hot_face == GSIS_HOT_TRANSPORT && o->synth_form != 0)
    return fail(ctx, GSIS_E_UNSUPPORTED,
                "options.synth_form 1 needs central HoT faces (options.hot_face 0)");
  HIPCHK(ctx, hipSetDevice(ctx->device));

  gsis_plan *pl = new gsis_plan;
  pl->ctx = ctx;
  pl->stream = (hipStream_t)o->stream;
  pl->device_ptrs = o->device_ptrs;
  pl->profile = arena ? 0 : o->profile;
  pl->arena = arena;
  pl->arena_cap = arena_cap;
  pl->pseudo = (o->cfl_p > 0 || o->beta > 0) ? 1 : 0;
  PlanDev &P = pl->P;
  const int nx = p->nx, ny = p->ny, N = nx * ny, K = p->K;
  P.nx = nx; P.ny = ny; P.N = N; P.K = K; P.nbf = 2 * (nx + ny);
  P.dx = p->dx; P.dy = p->dy; P.V = p->dx * p->dy;
  P.method = o->method; P.precision = o->precision; P.order = o->order;
  P.limiter = o->limiter ? 1 : 0; P.alsm = o->alsm ? 1 : 0; P.hot_face = o->hot_face;
  P.tol = o->tol; P.max_iter = o->max_iter; P.synth_rtol = o->synth_rtol;
  P.synth_max_iter = o->synth_max_iter;
  P.synth_form = o->method == GSIS_GSIS ? o->synth_form : 0;
  P.synth_sub = o->synth_sub;
  if (mt) {
    P.td = 1;
    P.sub_iter = mt->sub_iter;
    P.tdiag = 1.0 / (mt->c * mt->dt);
    P.ca = mt->a * mt->c;
    P.dt = mt->dt;
  }
  auto bail = [&](gsis_status s) {
    if (full) *full = pl->arena_full;
    gsis_plan_destroy(pl);
    return s;
  };

  // -- regroup ordinates by quadrant (bit 0: mu < 0, bit 1: eta < 0)
  pl->perm.clear();
  for (int qd = 0; qd < 4; ++qd) {
    P.qoff[qd] = (int)pl->perm.size();
    for (int k = 0; k < K; ++k) {
      int qk = (mu[k] < 0 ? 1 : 0) | (eta[k] < 0 ? 2 : 0);
      if (qk == qd) pl->perm.push_back(k);
    }
    P.Kq[qd] = (int)pl->perm.size() - P.qoff[qd];
  }
  P.qoff[4] = K;
  std::vector<double> amu(K), aeta(K), wv(K), wmu(K), weta(K);
  pl->swmu = pl->sweta = 0;
  for (int kk = 0; kk < K; ++kk) {
    const int k = pl->perm[kk];
    amu[kk] = std::fabs(mu[k]) / p->dx;
    aeta[kk] = std::fabs(eta[k]) / p->dy;
    wv[kk] = w[k];
    wmu[kk] = w[k] * mu[k];
    weta[kk] = w[k] * eta[k];
    pl->swmu += wmu[kk];
    pl->sweta += weta[kk];
    P.sw += wv[kk];
  }
  P.swm = pl->swmu;
  P.swe = pl->sweta;
  const bool f32 = P.precision == GSIS_FP32_MIXED;

  {
    // transport step: 0 residual kernel + recurrence, 3 pipelined (one
    // launch); 1 two-kernel reference and 2 fused wavefront sweep (tests
    // compare them); GSIS_SWEEP_REFERENCE=0..3 picks one. By default the
    // pipelined step runs FP64 problems of at least 2^26 cell-ordinates,
    // where enough rows run at once to hide its longer step (1024 x 1024 x
    // 128: 1.46 against 1.74 ms); on smaller grids the wavefront's length
    // decides and the split step is faster (256 x 256 x 128: 0.20 against
    // 0.13 ms), as it is in FP32-mixed form.
    const char *e = getenv("GSIS_SWEEP_REFERENCE");
    if (e && e[0] >= '0' && e[0] <= '3' && e[1] == 0)
      P.sweep_impl = e[0] - '0';
    else
      P.sweep_impl = (!f32 && (long long)N * K >= (1LL << 26)) ? 3 : 0;
    // the time terms live in the residual kernels of the split and
    // pipelined steps only
    if (P.td && P.sweep_impl != 3) P.sweep_impl = 0;
  }
  {
    // pipelined step: bands of 64 rows per workgroup (GSIS_PIPE_BANDS=1, 2
    // or 4 sets it), parts to cover the rows
    int nb = 2;
    const char *e = getenv("GSIS_PIPE_BANDS");
    if (e && (e[0] == '1' || e[0] == '2' || e[0] == '4') && e[1] == 0) nb = e[0] - '0';
    P.pipe_bands = nb;
    P.pipe_parts = P.sweep_impl == 3 ? (ny + 64 * nb - 1) / (64 * nb) : 1;
  }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess)
    cus = 0;
  {
    // workgroups per ordinate in the recurrence (GSIS_CHAIN_PARTS=1..4 sets
    // it): parts of about 256 rows (one wave per SIMD), at most 4, each a
    // multiple of 64 rows and at most 1024, the top part not empty. A wave
    // outside its rows' steps costs nothing, and a hand-over through memory
    // costs 10 us or so whatever the width, so up to 384 rows stay in one
    // workgroup where that is less than what five or six waves on four SIMDs
    // lose: in FP32-mixed form always, in FP64 on grids that are not wide.
    // An iteration (SI, FP64), 1 part and 2: 256 rows x 128 ordinates 133 and
    // 146 us; 300 rows, 32 ordinates: 512 wide 182 and 187, 768 wide 245 and
    // 242, 1536 wide 546 and 496; 384 rows, 64 ordinates: 384 wide 185 and 188,
    // 512 wide 265 and 246, 1536 wide 731 and 654; 12 ordinates the same way
    // (384 x 1536 575 and 503, 256 x 256 104 and 117), 256 rows of any width
    // one part (4096 x 12 972 and 989). FP32-mixed 384 x 1024 x 12 292 and 318.
    // Above: 400 rows, 128 ordinates 359 and 355; 512, 128: 546 and 531 (3:
    // 532); 700, 64: 665 and 627 (3: 583); 1000, 16: 1088 and 990 (4: 840). Few
    // ordinates are no reason for more parts: 512 rows, 4 ordinates 280 us in
    // 2, 284 in 4.
    const int waves = (ny + 63) / 64;
    const bool one = ny <= 384 && (waves <= 4 || f32 || (waves - 4) * nx <= 768);
    int parts = one ? 1 : std::min((ny + 255) / 256, 4);
    // the adjoint's sweep loads twice as much a step: parts of about 128 rows,
    // two waves, but one part on grids too narrow to earn the hand-overs. A pass
    // (SI) at 32 ordinates, 1 part and this rule's number otherwise: 192 rows x
    // 96 columns 73.5 and 81.3 us, x 512 145.7 and 147.5 (2), x 1024 equal;
    // 256 x 96 84.5 and 90.1 (2), x 256 119.9 and 118.3, x 512 178 and 167; 512 x
    // 96 120 and 136 (4), x 160 148 and 151, x 256 188 and 175; 1024 x 96 204 and
    // 228 (4), x 160 258 and 254. 128 ordinates likewise (512 x 96 139 and 157, x
    // 512 609 and 542).
    const int narrow = ny <= 192 ? 512 : ny <= 256 ? 224 : ny <= 512 ? 160 : 128;
    int aparts = nx <= narrow ? 1 : std::min((ny + 127) / 128, 4);
    const char *e = getenv("GSIS_CHAIN_PARTS");
    if (e && e[0] >= '1' && e[0] <= '4' && e[1] == 0) parts = aparts = e[0] - '0';
    auto split = [&](int n, int &np, int &rows) {
      np = std::max(1, std::min(n, 4));
      rows = 0;
      for (; np > 1; --np) {
        rows = ((ny + np - 1) / np + 63) / 64 * 64;
        if (rows <= 1024 && (np - 1) * rows < ny) break;
      }
      if (np <= 1) rows = 0;
    };
    if (!arena) split(aparts, P.adj_parts, P.adj_rows);   // (no adjoint there)
    if (P.sweep_impl == 1 || P.sweep_impl == 2) parts = 1;
    split(parts, P.chain_parts, P.chain_rows);
  }
  P.mom_split = moment_split(P);
  P.mom_parts = lean ? 1 : P.mom_split;
  // residual tiles (GSIS_RESID_DIAGONALS=3, 7, .. 59 sets their length)
  P.resid_rd = residual_tile_diagonals(nx, ny, residual_pairs(P), share, cus);
  {
    const char *e = getenv("GSIS_RESID_DIAGONALS");
    const int rd = e ? atoi(e) : 0;
    if (rd >= 3 && rd <= kMaxResidDiagonals && rd % 4 == 3 && std::to_string(rd) == e) P.resid_rd = rd;
  }
  if (lean && residual_tiles(nx, ny, 31).size() < residual_tiles(nx, ny, P.resid_rd).size())
    P.resid_rd = 31;
  const std::vector<int2> rtiles = residual_tiles(nx, ny, P.resid_rd);
  P.n_rtiles = (int)rtiles.size();
  // partial sums of w r^2: one per residual wave
  P.n_tres = P.sweep_impl == 3 ? K * P.pipe_parts * P.pipe_bands
                               : P.n_rtiles * residual_pairs(P);

  // -- device arrays
  Pack pack;
  pack.add(&P.amu, amu);
  pack.add(&P.aeta, aeta);
  pack.add(&P.w, wv);
  pack.add(&P.wmu, wmu);
  pack.add(&P.weta, weta);
  pack.add(&P.rtiles, rtiles);
  pack.add(&P.dso, diag_row0_table(nx, ny));
  if (f32) {
    // w, w mu, w eta in FP32 for the moment sums of the deviations
    std::vector<float> wf(3 * (size_t)K);
    for (int kk = 0; kk < K; ++kk) {
      wf[kk] = (float)wv[kk];
      wf[K + kk] = (float)wmu[kk];
      wf[2 * K + kk] = (float)weta[kk];
    }
    pack.add(&P.w_f, wf);
  }
  // for the set-up alone; in the caller's region inside arrays not in use yet
  int *perm = nullptr;
  unsigned long long *bad = nullptr;
  if (!arena) {
    pack.add(&perm, pl->perm);
    pack.add(&bad, std::vector<unsigned long long>(3, ~0ull));
  }
  MGLevel L0;
  L0.nx = nx;
  L0.ny = ny;
  const size_t nbk = (size_t)P.nbf * K;
  if ((st = alloc_intensity(pl, 0, (size_t)N * K, f32)) ||
      (st = alloc_intensity(pl, 1, (size_t)N * K, f32)) ||
      (st = dalloc(pl, &P.R, P.sweep_impl == 1 ? (size_t)N * K : 1)) ||
      (st = dalloc(pl, &P.cellq, (size_t)4 * N * 6)) || (st = dalloc(pl, &P.dynq, (size_t)4 * N * 3)) ||
      (st = dalloc(pl, &P.rowbuf, (size_t)K * 3 * nx)) || (st = dalloc(pl, &P.sdq, (size_t)4 * N)) ||
      (st = dalloc(pl, &P.sig_t, N)) || (st = dalloc(pl, &P.sig_a, N)) ||
      (st = dalloc(pl, &P.sig_s, N)) || (st = dalloc(pl, &P.q, N)) ||
      (st = dalloc(pl, &P.cE, N)) || (st = dalloc(pl, &P.cW, N)) ||
      (st = dalloc(pl, &P.cN, N)) || (st = dalloc(pl, &P.cS, N)) ||
      (st = dalloc(pl, &P.src, N)) || (st = dalloc(pl, &P.phi, N)) ||
      (st = dalloc(pl, &P.phih, N)) || (st = dalloc(pl, &P.Fx, N)) ||
      (st = dalloc(pl, &P.mom_part, (size_t)12 * P.mom_parts * N)) ||
      (st = dalloc(pl, &P.Fy, N)) || (st = dalloc(pl, &P.delta, N)) ||
      (st = dalloc(pl, &P.hx, N)) || (st = dalloc(pl, &P.hy, N)) ||
      (st = dalloc(pl, &P.rhs, N)) || (st = dalloc(pl, &P.bnd, nbk)) ||
      (st = dalloc(pl, &P.bflux, P.nbf)) || (st = dalloc(pl, &P.kappa, P.nbf)) ||
      (st = dalloc(pl, &P.err_hist, o->max_iter)) ||
      (st = dalloc(pl, &P.tres_hist, o->max_iter)) ||
      (st = dalloc(pl, &P.tres_part, tres_slots(P))) ||
      (st = dalloc(pl, &P.src2_part, (size_t)(N + 255) / 256)) ||
      (st = dalloc(pl, &P.state, kStateWords)) || (st = dalloc(pl, &P.last_err, 2)) ||
      (st = dalloc(pl, &P.err_parts, 2 * (size_t)((N + 255) / 256) + 2)) ||
      (st = alloc_level(pl, L0)))
    return bail(st);
  if (hand_parts(P) > 1 && (st = dalloc(pl, &P.hand, (size_t)K * (hand_parts(P) - 1) * nx)))
    return bail(st);
  if (f32 && ((st = dalloc(pl, &P.sdq_f, (size_t)4 * N)) || (st = dalloc(pl, &P.base, N))))
    return bail(st);
  if (!f32) P.base = P.delta;
  if (P.method == GSIS_GSIS && P.hot_face == GSIS_HOT_TRANSPORT &&
      (st = dalloc(pl, &P.ftp, (size_t)8 * N)))
    return bail(st);
  if (P.td &&
      ((st = dalloc(pl, &P.cv, N)) || (st = dalloc(pl, &P.T0, N)) || (st = dalloc(pl, &P.Tm, N)) ||
       (st = dalloc(pl, &P.Tn, N)) || (st = dalloc(pl, &P.Tsub0, N)) ||
       (st = dalloc(pl, &P.Tsub1, N)) || (st = dalloc(pl, &P.rho_n, N)) ||
       (st = dalloc(pl, &P.err_parts_T, 2 * (size_t)((N + 255) / 256) + 2)) ||
       (st = dalloc(pl, &P.In, (size_t)N * K))))
    return bail(st);
  P.mg.assign(1, L0);

  // -- the caller's fields, checked on the device. Work the caller has on the
  // default stream comes first, as it would for a blocking copy
  hipStream_t s = pl->stream;
  if (hipStreamSynchronize(nullptr) != hipSuccess)
    return bail(fail(ctx, GSIS_E_DEVICE, "hipStreamSynchronize failed"));
  if ((st = pack.commit(pl)) || (st = fetch_dev(pl, p->sigma_a, P.sig_a, N, "sigma_a")) ||
      (st = fetch_dev(pl, p->sigma_s, P.sig_s, N, "sigma_s")) ||
      (st = fetch_dev(pl, p->q, P.q, N, "q")))
    return bail(st);
  if (P.td && ((st = fetch_dev(pl, mt->cv, P.cv, N, "material.cv")) ||
               (st = fetch_dev(pl, mt->T0, P.T0, N, "material.T0"))))
    return bail(st);
  if (arena) {
    perm = (int *)P.rowbuf;
    bad = (unsigned long long *)P.mom_part;
    if (hipMemcpyAsync(perm, pl->perm.data(), K * sizeof(int), hipMemcpyHostToDevice, s) !=
            hipSuccess ||
        hipMemsetAsync(bad, 0xff, 3 * sizeof *bad, s) != hipSuccess)
      return bail(fail(ctx, GSIS_E_DEVICE, "preparing the checks of the problem failed"));
  }
  launch_check_cells(N, P.sig_a, P.sig_s, P.q, P.cv, P.T0, P.sig_t, bad, s);
  const double *bnd_h = nullptr;   // bnd_in where the host checks it
  std::vector<double> bnd_copy;
  if (!p->bnd_in) {
    if (hipMemsetAsync(P.bnd, 0, nbk * sizeof(double), s) != hipSuccess)
      return bail(fail(ctx, GSIS_E_DEVICE, "hipMemsetAsync failed"));
  } else if (o->device_ptrs && kernel_reaches(ctx, p->bnd_in)) {
    launch_setup_bnd(nbk, K, p->bnd_in, perm, P.bnd, bad, s);
  } else {
    std::vector<double> bnd(nbk);
    bnd_h = p->bnd_in;
    if (o->device_ptrs) {
      if ((st = fetch(ctx, p->bnd_in, nbk, 1, bnd_copy, "bnd_in"))) return bail(st);
      bnd_h = bnd_copy.data();
    }
    for (size_t t = 0; t < nbk; ++t) {
      const size_t fc = t / K;
      bnd[t] = bnd_h[fc * K + pl->perm[t - fc * K]];
    }
    // (checked below with the caller's index, after the cells)
    if (hipMemcpyAsync(P.bnd, bnd.data(), nbk * sizeof(double), hipMemcpyHostToDevice, s) !=
            hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return bail(fail(ctx, GSIS_E_DEVICE, "copying bnd_in failed"));
  }
  {
    unsigned long long hb[3];
    if (hipMemcpyAsync(hb, bad, sizeof hb, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return bail(fail(ctx, GSIS_E_DEVICE, "reading the problem's fields: %s",
                       hipGetErrorString(hipGetLastError())));
    if (bnd_h)
      for (size_t t = 0; t < nbk && hb[1] == ~0ull; ++t)
        if (!std::isfinite(bnd_h[t])) hb[1] = t;
    for (int k = 0; k < 3; k += 2) {
      if (hb[k] == ~0ull) continue;
      const size_t c = hb[k] >> 3;
      const char *const what[] = {"sigma_a[%zu] must be finite and >= 0",
                                  "sigma_s[%zu] must be finite and >= 0",
                                  "sigma_a[%zu] + sigma_s[%zu] must be > 0", "q[%zu] is not finite",
                                  "material.cv[%zu] must be finite and > 0",
                                  "material.T0[%zu] must be finite and >= 0"};
      if (k == 2 && hb[1] != ~0ull) break;
      return bail(fail(ctx, GSIS_E_INVALID_ARG, what[hb[k] & 7], c, c));
    }
    if (hb[1] != ~0ull)
      return bail(fail(ctx, GSIS_E_INVALID_ARG, "bnd_in[%zu][%zu] is not finite",
                       (size_t)hb[1] / K, (size_t)hb[1] % K));
  }

  // -- coefficients, records and the level-0 operator
  {
    SetupArgs a;
    a.nx = nx; a.ny = ny; a.alsm = P.alsm;
    a.dx = P.dx; a.dy = P.dy; a.V = P.V; a.tdiag = P.tdiag;
    a.cfl_p = o->cfl_p; a.beta = o->beta; a.dref = std::min(p->dx, p->dy);
    a.st = P.sig_t; a.sa = P.sig_a;
    a.cE = P.cE; a.cW = P.cW; a.cN = P.cN; a.cS = P.cS; a.kappa = P.kappa;
    a.diag = L0.diag; a.ax = L0.ax; a.ay = L0.ay;
    a.cellq = P.cellq; a.sdq = P.sdq; a.sdq_f = P.sdq_f;
    launch_setup_cells(a, s);
  }
  // -- warm start
  if (o->I0) {
    std::vector<double> phi0(N, 0.0);
    std::vector<double> I0;
    if ((st = fetch(ctx, o->I0, (size_t)N * K, o->device_ptrs, I0, "I0"))) return bail(st);
    pl->I0_host.assign((size_t)N * K, 0.0);
    for (int kk = 0; kk < K; ++kk) {
      const int k = pl->perm[kk];
      const int qd = (mu[k] < 0 ? 1 : 0) | (eta[k] < 0 ? 2 : 0);
      for (int j = 0; j < ny; ++j)
        for (int i = 0; i < nx; ++i) {
          const int xl = (qd & 1) ? nx - 1 - i : i, yl = (qd & 2) ? ny - 1 - j : j;
          pl->I0_host[(size_t)kk * N + dg_idx(xl, yl, nx, ny)] = I0[(size_t)(j * nx + i) * K + k];
        }
    }
    for (int c = 0; c < N; ++c) {
      double s = 0;
      for (int k = 0; k < K; ++k) s += w[k] * I0[(size_t)c * K + k];
      phi0[c] = s;
    }
    if (f32) {
      // stored deviation from phi0/(4 pi); the first read adds base = phi0
      pl->I0_host_f.resize((size_t)N * K);
      for (int kk = 0; kk < K; ++kk) {
        const int k = pl->perm[kk];
        const int qd = (mu[k] < 0 ? 1 : 0) | (eta[k] < 0 ? 2 : 0);
        for (int j = 0; j < ny; ++j)
          for (int i = 0; i < nx; ++i) {
            const int xl = (qd & 1) ? nx - 1 - i : i, yl = (qd & 2) ? ny - 1 - j : j;
            const int c = j * nx + i;
            pl->I0_host_f[(size_t)kk * N + dg_idx(xl, yl, nx, ny)] =
                (float)(I0[(size_t)c * K + k] - phi0[c] / kFourPi);
          }
      }
      pl->I0_host.clear();
    }
    if (arena) {   // hx is free until the first iteration, and the only reset is below
      P.phi0 = P.hx;
      if (hipMemcpy(P.phi0, phi0.data(), N * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)
        return bail(fail(ctx, GSIS_E_DEVICE, "copying the warm start failed"));
    } else if ((st = upload(pl, &P.phi0, phi0))) {
      return bail(st);
    }
  }
  if ((st = setup_synth(pl, P))) return bail(st);
  if ((st = make_single_set(pl))) return bail(st);
  if (arena) {
    // pageable host flags: the synthetic solve's copies of them are followed
    // by a stream synchronisation either way
    pl->host_scal = pl->host_flag_store;
  } else {
    // flags read back by the synthetic solve: [0, 3) state and [8] the CG
    // count of the last forward solve; [4, 7) and [12] the same for the
    // adjoint's solves
    void *h = nullptr;
    hipError_t e = hipHostMalloc(&h, kHostScal * sizeof(double), hipHostMallocDefault);
    if (e != hipSuccess) return bail(fail(ctx, GSIS_E_OOM, "hipHostMalloc: %s", hipGetErrorString(e)));
    memset(h, 0, kHostScal * sizeof(double));
    pl->host_scal = (double *)h;
    if ((e = hipEventCreateWithFlags(&pl->spec_ev, hipEventDisableTiming)) != hipSuccess) {
      pl->spec_ev = nullptr;
      return bail(fail(ctx, GSIS_E_DEVICE, "hipEventCreate: %s", hipGetErrorString(e)));
    }
  }
  if ((st = gsis_plan_reset(pl))) return bail(st);
  *out = pl;
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_create(gsis_ctx *ctx, const gsis_problem *p,
                                        const gsis_options *o, gsis_plan **out) {
  return plan_create(ctx, p, o, out, nullptr, 0);
}

gsis_status plan_create_shared(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                               int share, gsis_plan **out) {
  return plan_create(ctx, p, o, out, nullptr, 0, nullptr, share);
}

extern "C" void gsis_plan_destroy(gsis_plan *pl) {
  if (!pl) return;
  if (pl->stream) (void)hipStreamSynchronize(pl->stream);
  else (void)hipDeviceSynchronize();
  for (void *v : pl->allocs) (void)hipFree(v);
  for (hipEvent_t e : pl->events) (void)hipEventDestroy(e);
  if (pl->spec_ev) (void)hipEventDestroy(pl->spec_ev);
  adjoint_release(pl);
  if (pl->host_scal && !pl->arena) (void)hipHostFree(pl->host_scal);
  delete pl;
}

gsis_status plan_reset_enqueue(gsis_plan *pl) {
  gsis_ctx *ctx = pl->ctx;
  PlanDev &P = pl->P;
  const size_t NK = (size_t)P.N * P.K;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  hipStream_t s = pl->stream;
  const bool f32 = P.precision == GSIS_FP32_MIXED;
  if (f32 && !pl->I0_host_f.empty())
    HIPCHK(ctx, hipMemcpyAsync(P.I[0], pl->I0_host_f.data(), NK * sizeof(float),
                               hipMemcpyHostToDevice, s));
  else if (!f32 && !pl->I0_host.empty())
    HIPCHK(ctx, hipMemcpyAsync(P.I[0], pl->I0_host.data(), NK * sizeof(double),
                               hipMemcpyHostToDevice, s));
  else
    HIPCHK(ctx, hipMemsetAsync(P.I[0], 0, NK * (f32 ? sizeof(float) : sizeof(double)), s));
  launch_plan_reset(P, tres_slots(P), s);
  launch_source(P.S, s);
  HIPCHK(ctx, hipGetLastError());
  pl->prof_iters = 0;
  pl->ahead = 0;
  pl->ahead_pending = pl->ended = false;
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_reset(gsis_plan *pl) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_status st = plan_reset_enqueue(pl);
  if (st) return st;
  HIPCHK(pl->ctx, hipStreamSynchronize(pl->stream));
  return GSIS_OK;
}

static gsis_status record(gsis_plan *pl, int slot) {
  if (!pl->profile) return GSIS_OK;
  const size_t idx = (size_t)pl->prof_iters * (GSIS_NUM_PHASES + 1) + slot;
  while (pl->events.size() <= idx) {
    hipEvent_t e;
    HIPCHK(pl->ctx, hipEventCreate(&e));
    pl->events.push_back(e);
  }
  HIPCHK(pl->ctx, hipEventRecord(pl->events[idx], pl->stream));
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_iterate(gsis_plan *pl, int32_t n) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  if (n < 0) return fail(ctx, GSIS_E_INVALID_ARG, "n must be >= 0");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  PlanDev &P = pl->P;
  hipStream_t s = pl->stream;
  gsis_status st;
  // GSIS plans whose synthetic solve is one kernel do not wait for it. The done
  // flag is copied to the host after 2 kRunAhead iterations, counted over the
  // calls, and every kRunAhead further ones, and each copy is looked at when the
  // next is due: the host never is more than three times that many ahead of the
  // device or past the end of the solve, and the device never runs dry for the
  // look. 32 x 32, S4, copies every 4, 8 and 16: 44.4, 43.9 and 43.5 us an
  // iteration, and 1.64, 1.75 and 1.98 ms for a call for 1000 of which the solve
  // takes 33; the first copy is late because a call for 9 iterations pays 1 % for
  // it.
  const bool ahead = P.method == GSIS_GSIS && synth_in_one_kernel(P.S) && pl->spec_ev;
  if (ahead && pl->ended) return GSIS_OK;   // the iterations would do no work
  for (int it = 0; it < n; ++it) {
    int32_t *host_flag = (int32_t *)pl->host_scal;
    if (ahead && pl->ahead++ == (pl->ahead_pending ? 1 : 2) * kRunAhead) {
      if (pl->ahead_pending) {
        HIPCHK(ctx, hipEventSynchronize(pl->spec_ev));
        if (host_flag[kAheadFlag] != 0) {
          pl->ended = true;
          break;
        }
      }
      HIPCHK(ctx, hipMemcpyAsync(host_flag + kAheadFlag, P.state + 1, sizeof(int32_t),
                                 hipMemcpyDeviceToHost, s));
      HIPCHK(ctx, hipEventRecord(pl->spec_ev, s));
      pl->ahead_pending = true;
      pl->ahead = 1;
    }
    if (pl->profile && pl->prof_iters >= 100000) pl->profile = 0;
    if ((st = record(pl, 0))) return st;
    launch_residual(P, s);
    if ((st = record(pl, 1))) return st;
    launch_sweep(P, s);
    if ((st = record(pl, 2))) return st;
    // source iteration's update takes the moments from their partials itself
    // (the phase-timed pass keeps the combine with the moments)
    const bool fused = P.method != GSIS_GSIS && !P.td && P.precision == GSIS_FP64 && !pl->profile;
    launch_moments(P, s, P.method == GSIS_GSIS, !fused);
    if ((st = record(pl, 3))) return st;
    if (P.method == GSIS_GSIS) {
      launch_hot(P.S, s, P.mom_parts == 1);
    }
    if ((st = record(pl, 4))) return st;
    // the synthetic solve copies the device flags to the host once while it
    // runs (host_flag[0]: the outer iteration's done flag); cleared first,
    // so a nonzero value below was read during this iteration
    host_flag[0] = 0;
    bool updated = false;
    if (P.td) {
      // time-dependent form: sub-iterations of the material equation and
      // (GSIS) the synthetic equation, each from the previous sub-iterate
      for (int sub = 0; sub < P.sub_iter; ++sub) {
        launch_material(P.S, s, sub);
        if (P.method == GSIS_GSIS) {
          launch_synth_solve(P.S, s, host_flag, sub == 0 ? 1 : 3, sub);
          if (host_flag[0] != 0) break;
        }
      }
    } else if (P.method == GSIS_GSIS && P.synth_form == 1) {
      // face-averaged balance: sub-iterations from phi^{m+1/2}
      for (int sub = 0; sub < P.synth_sub; ++sub) {
        launch_wide_grad(P.S, s, sub == 0);
        launch_synth_solve(P.S, s, host_flag, 2);
        if (host_flag[0] != 0) break;
      }
    } else if (P.method == GSIS_GSIS) {
      // (the phase-timed pass keeps the update after the wait)
      updated = launch_synth_solve(P.S, s, host_flag, 1, 0, pl->profile ? nullptr : pl->spec_ev);
    }
    if ((st = record(pl, 5))) return st;
    if (!updated) launch_update(P.S, s, 0, fused ? P.mom_parts : 0);
    if ((st = record(pl, 6))) return st;
    HIPCHK(ctx, hipGetLastError());
    if (pl->profile) pl->prof_iters++;
    // an earlier iteration ended the solve (converged, diverged or at the
    // iteration cap): the remaining ones would only launch kernels that exit
    if (host_flag[0] != 0) break;
  }
  return GSIS_OK;
}

// Enqueues the copies of the flags and Err to the host (status_get reads them
// after a wait for the stream).
static gsis_status status_enqueue(gsis_plan *pl) {
  double *h = pl->host_scal + kStatusSlot;
  HIPCHK(pl->ctx, hipMemcpyAsync(h, pl->P.last_err, sizeof(double), hipMemcpyDeviceToHost,
                                 pl->stream));
  HIPCHK(pl->ctx, hipMemcpyAsync(h + 1, pl->P.state, 5 * sizeof(int32_t), hipMemcpyDeviceToHost,
                                 pl->stream));
  return GSIS_OK;
}
static gsis_status status_get(gsis_plan *pl, int32_t *n_iter, int32_t *converged,
                              double *last_err) {
  const double *h = pl->host_scal + kStatusSlot;
  int32_t stv[5];
  memcpy(stv, h + 1, sizeof stv);
  pl->ahead = 0;               // the stream is empty
  pl->ahead_pending = false;
  pl->ended = stv[1] != 0;
  if (stv[4] != 0)
    return fail(pl->ctx, GSIS_E_DEVICE,
                "the recurrence's workgroups of one ordinate stopped waiting for each other; "
                "reset the plan");
  if (n_iter) *n_iter = stv[0];
  if (converged) *converged = stv[1] == 1 ? 1 : (stv[1] == -1 ? -1 : 0);
  if (last_err) *last_err = h[0];
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_status(gsis_plan *pl, int32_t *n_iter, int32_t *converged,
                                        double *last_err) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  gsis_status st = status_enqueue(pl);
  if (st) return st;
  HIPCHK(ctx, hipStreamSynchronize(pl->stream));
  return status_get(pl, n_iter, converged, last_err);
}

extern "C" gsis_status gsis_plan_read(gsis_plan *pl, gsis_result *r) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  if (!r) return fail(ctx, GSIS_E_INVALID_ARG, "result is NULL");
  if (!r->phi || !r->Fx || !r->Fy) return fail(ctx, GSIS_E_INVALID_ARG, "result.phi/Fx/Fy is NULL");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  PlanDev &P = pl->P;
  hipStream_t s = pl->stream;
  int32_t n_iter = 0, conv = 0;
  double le = 0;
  gsis_status st = status_enqueue(pl);
  if (st) return st;
  // F of the final iterate: F_half plus the pending correction's flux; for
  // host memory staged in hx, hy, which are free here
  bool direct = pl->device_ptrs;
  for (const double *out : {r->phi, r->Fx, r->Fy, r->err_hist, r->tres_hist})
    direct = direct && kernel_reaches(ctx, out);
  if (direct)
    launch_plan_read(P, pl->swmu, pl->sweta, r->phi, r->Fx, r->Fy, r->err_hist, r->tres_hist, s);
  else
    launch_plan_read(P, pl->swmu, pl->sweta, nullptr, P.hx, P.hy, nullptr, nullptr, s);
  HIPCHK(ctx, hipGetLastError());
  HIPCHK(ctx, hipStreamSynchronize(s));
  if ((st = status_get(pl, &n_iter, &conv, &le))) return st;
  if (!direct) {
    const size_t bytes = P.N * sizeof(double);
    const hipMemcpyKind k = pl->device_ptrs ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    HIPCHK(ctx, hipMemcpyAsync(r->phi, P.phi, bytes, k, s));
    HIPCHK(ctx, hipMemcpyAsync(r->Fx, P.hx, bytes, k, s));
    HIPCHK(ctx, hipMemcpyAsync(r->Fy, P.hy, bytes, k, s));
    if (r->err_hist && n_iter > 0)
      HIPCHK(ctx, hipMemcpyAsync(r->err_hist, P.err_hist, n_iter * sizeof(double), k, s));
    if (r->tres_hist && n_iter > 0)
      HIPCHK(ctx, hipMemcpyAsync(r->tres_hist, P.tres_hist, n_iter * sizeof(double), k, s));
    HIPCHK(ctx, hipStreamSynchronize(s));
  }
  r->n_iter = n_iter;
  r->final_err = n_iter > 0 ? le : INFINITY;
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_transport_form(gsis_plan *pl, int32_t *form, int32_t *bands,
                                                int32_t *parts) {
  if (!pl) return GSIS_E_INVALID_ARG;
  if (!form) return fail(pl->ctx, GSIS_E_INVALID_ARG, "form is NULL");
  const PlanDev &P = pl->P;
  *form = P.sweep_impl;
  if (bands) *bands = P.sweep_impl == 3 ? P.pipe_bands : 0;
  if (parts) *parts = P.sweep_impl == 3 ? P.pipe_parts : P.chain_parts;
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_synth_vcycles(gsis_plan *pl, int64_t *vcycles) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  if (!vcycles) return fail(ctx, GSIS_E_INVALID_ARG, "vcycles is NULL");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  double v = 0;
  HIPCHK(ctx, hipMemcpyAsync(&v, synth_vcycle_total(pl->P), sizeof v, hipMemcpyDeviceToHost,
                             pl->stream));
  HIPCHK(ctx, hipStreamSynchronize(pl->stream));
  *vcycles = (int64_t)v;
  return GSIS_OK;
}

extern "C" gsis_status gsis_plan_phase_times(gsis_plan *pl, double *ms, int32_t *n_iter) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  if (!ms) return fail(ctx, GSIS_E_INVALID_ARG, "ms is NULL");
  HIPCHK(ctx, hipStreamSynchronize(pl->stream));
  for (int ph = 0; ph < GSIS_NUM_PHASES; ++ph) ms[ph] = 0;
  for (int it = 0; it < pl->prof_iters; ++it)
    for (int ph = 0; ph < GSIS_NUM_PHASES; ++ph) {
      float t = 0;
      const size_t e0 = (size_t)it * (GSIS_NUM_PHASES + 1) + ph;
      HIPCHK(ctx, hipEventElapsedTime(&t, pl->events[e0], pl->events[e0 + 1]));
      ms[ph] += t;
    }
  if (n_iter) *n_iter = pl->prof_iters;
  pl->prof_iters = 0;
  return GSIS_OK;
}

// Plan, iterate until Err < tol, divergence or max_iter, read, destroy.
static gsis_status solve_with(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                              gsis_result *r, char *arena, size_t arena_cap) {
  if (!ctx) return fail(nullptr, GSIS_E_INVALID_ARG, "ctx is NULL");
  if (!r) return fail(ctx, GSIS_E_INVALID_ARG, "result is NULL");
  gsis_plan *pl = nullptr;
  // a region too small for the form that runs fastest may hold the lean one
  // (the same fields, fewer partial sums kept)
  bool full = false;
  gsis_status st = plan_create(ctx, p, o, &pl, arena, arena_cap, nullptr, 1, false, &full);
  if (st && full) st = plan_create(ctx, p, o, &pl, arena, arena_cap, nullptr, 1, true);
  if (st) return st;
  int32_t n = 0, conv = 0;
  double le = 0;
  const int chunk = 8;
  while (true) {
    const int todo = std::min(chunk, o->max_iter - n);
    if ((st = gsis_plan_iterate(pl, todo))) break;
    if ((st = gsis_plan_status(pl, &n, &conv, &le))) break;
    if (conv != 0 || n >= o->max_iter) break;
  }
  if (st == GSIS_OK) st = gsis_plan_read(pl, r);
  gsis_plan_destroy(pl);
  if (st) return st;
  if (conv == -1) return GSIS_DIVERGED;
  if (conv == 0) return GSIS_NOT_CONVERGED;
  return GSIS_OK;
}

extern "C" gsis_status gsis_solve(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                                  gsis_result *r) {
  return solve_with(ctx, p, o, r, nullptr, 0);
}

// ------------------------------------------------------ solve without allocation
// The device state of gsis_solve_noalloc lives in this file-scope array (one
// copy per GPU, held until the process ends). In host code its name only
// stands in for the symbol: the device address of each GPU's copy comes from
// hipGetSymbolAddress, taken once per device with that device current.
constexpr size_t kScratchBytes = (size_t)256 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxScratchDevices] = {};

// Device address of this device's scratch copy (the context's device is
// current).
gsis_status scratch_address(gsis_ctx *ctx, char **out) {
  if (ctx->device < 0 || ctx->device >= kMaxScratchDevices)
    return fail(ctx, GSIS_E_UNSUPPORTED, "gsis_solve_noalloc: device %d beyond %d", ctx->device,
                kMaxScratchDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[ctx->device]) {
    void *ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(ctx, GSIS_E_DEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_scratch_ptr[ctx->device] = ptr;
  }
  *out = (char *)g_scratch_ptr[ctx->device];
  return GSIS_OK;
}
}  // namespace

extern "C" gsis_status gsis_solve_noalloc(gsis_ctx *ctx, const gsis_problem *p,
                                          const gsis_options *o, gsis_result *r) {
  if (!ctx) return fail(nullptr, GSIS_E_INVALID_ARG, "ctx is NULL");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  char *base = nullptr;
  gsis_status st = scratch_address(ctx, &base);
  if (st) return st;
  return solve_with(ctx, p, o, r, base, kScratchBytes);
}

// ------------------------------------------------------- time-dependent form
extern "C" gsis_status gsis_td_create(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                                      const gsis_material *mt, gsis_plan **out) {
  if (!mt) return fail(ctx, GSIS_E_INVALID_ARG, "material is NULL");
  return plan_create(ctx, p, o, out, nullptr, 0, mt);
}

extern "C" gsis_status gsis_td_advance(gsis_plan *pl, int32_t n_steps, int32_t *inner_iters,
                                       double *last_err) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  if (!pl->P.td) return fail(ctx, GSIS_E_INVALID_ARG, "not a time-dependent plan");
  if (n_steps < 0) return fail(ctx, GSIS_E_INVALID_ARG, "n_steps must be >= 0");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  gsis_status worst = GSIS_OK;
  for (int step = 0; step < n_steps; ++step) {
    launch_td_begin(pl->P, pl->stream);
    HIPCHK(ctx, hipGetLastError());
    pl->ahead = 0;
    pl->ahead_pending = pl->ended = false;
    int32_t n = 0, conv = 0;
    double le = 0;
    gsis_status st;
    while (true) {
      if ((st = gsis_plan_iterate(pl, std::min(8, pl->P.max_iter - n)))) return st;
      if ((st = gsis_plan_status(pl, &n, &conv, &le))) return st;
      if (conv != 0 || n >= pl->P.max_iter) break;
    }
    if (inner_iters) inner_iters[step] = n;
    if (last_err) last_err[step] = le;
    if (conv == -1) return GSIS_DIVERGED;
    if (conv == 0) worst = GSIS_NOT_CONVERGED;
  }
  return worst;
}

extern "C" gsis_status gsis_td_read(gsis_plan *pl, double *rho, double *T, double *Fx,
                                    double *Fy) {
  if (!pl) return GSIS_E_INVALID_ARG;
  gsis_ctx *ctx = pl->ctx;
  if (!pl->P.td) return fail(ctx, GSIS_E_INVALID_ARG, "not a time-dependent plan");
  if (!rho || !T || !Fx || !Fy) return fail(ctx, GSIS_E_INVALID_ARG, "an output is NULL");
  gsis_result r;
  std::memset(&r, 0, sizeof r);
  r.phi = rho; r.Fx = Fx; r.Fy = Fy;
  gsis_status st = gsis_plan_read(pl, &r);
  if (st) return st;
  const hipMemcpyKind k = pl->device_ptrs ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  HIPCHK(ctx, hipMemcpyAsync(T, pl->P.Tm, pl->P.N * sizeof(double), k, pl->stream));
  HIPCHK(ctx, hipStreamSynchronize(pl->stream));
  return GSIS_OK;
}
