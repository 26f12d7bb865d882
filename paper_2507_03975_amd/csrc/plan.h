// plan.h -- host-side state shared by the C-ABI translation units: the
// context and plan objects, error reporting, device allocation helpers and
// the synthetic-solve set-up.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "gsis_internal.h"

using namespace gsis;

struct gsis_ctx {
  int device = 0;
  std::string err;
};

constexpr int kHostScal = 16, kStatusSlot = 8;   // doubles
constexpr int kAheadFlag = 28;                   // int32: the done flag of an earlier iteration
constexpr int kRunAhead = 8;

struct gsis_plan {
  gsis_ctx *ctx = nullptr;
  PlanDev P;
  hipStream_t stream = nullptr;
  int device_ptrs = 0;
  int profile = 0;
  std::vector<int> perm;          // internal ordinate -> caller ordinate
  double swmu = 0, sweta = 0;     // sum_k w_k mu_k, sum_k w_k eta_k
  std::vector<double> I0_host;    // warm start in the internal layout (may be empty)
  std::vector<float> I0_host_f;   // FP32-mixed: I0 - phi0/(4 pi) in the internal layout
  std::vector<void *> allocs;
  char *slab = nullptr;           // the allocation small arrays are carved from
  size_t slab_used = 0, slab_cap = 0;
  double *host_scal = nullptr;    // pinned: the synthetic solves' flags, then
                                  // (kStatusSlot) the status read-out
  hipEvent_t spec_ev = nullptr;   // marks the synthetic solve's flag copy (see
                                  // launch_synth_solve); not in the allocation-free solve
  // plans whose synthetic solve is one kernel (gsis_plan_iterate): iterations
  // enqueued since the last look at the done flag, a copy of the flag is under
  // way, the solve was seen to have ended
  int ahead = 0;
  bool ahead_pending = false, ended = false;
  // profiling: per iteration GSIS_NUM_PHASES + 1 events bracketing the phases
  std::vector<hipEvent_t> events;
  int prof_iters = 0;
  int pseudo = 0;                 // a pseudo-time shift is on
  AdjointBuffers *adj = nullptr;  // adjoint state (first gsis_plan_adjoint)
  // device memory carved from a caller-free region instead of hipMalloc
  // (gsis_solve_noalloc): base, bytes used, capacity; the host flags then
  // live in host_flag_store instead of pinned memory
  char *arena = nullptr;
  size_t arena_used = 0, arena_cap = 0;
  bool arena_full = false;        // an array did not fit
  double host_flag_store[kHostScal] = {};
};

extern thread_local std::string g_create_err;

inline gsis_status fail_impl(gsis_ctx *ctx, gsis_status st, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (ctx) ctx->err = buf;
  else g_create_err = buf;
  return st;
}
#define fail fail_impl

#define HIPCHK(ctx, call)                                                             \
  do {                                                                                \
    hipError_t e_ = (call);                                                           \
    if (e_ != hipSuccess)                                                             \
      return fail(ctx, GSIS_E_DEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
  } while (0)


constexpr size_t kSlabShare = 1 << 20, kSlabBytes = 4 << 20;

template <typename T>
gsis_status dalloc(gsis_plan *pl, T **p, size_t n) {
  void *v = nullptr;
  if (pl->arena) {
    // 256-byte aligned pieces of the region, in allocation order
    const size_t bytes = (std::max<size_t>(n, 1) * sizeof(T) + 255) & ~(size_t)255;
    if (bytes > pl->arena_cap - pl->arena_used) {
      pl->arena_full = true;
      return fail(pl->ctx, GSIS_E_INVALID_ARG,
                  "the problem needs more device memory than the %zu-byte scratch region of "
                  "gsis_solve_noalloc (%zu bytes used when %zu more were asked for)",
                  pl->arena_cap, pl->arena_used, bytes);
    }
    *p = (T *)(pl->arena + pl->arena_used);
    pl->arena_used += bytes;
    return GSIS_OK;
  }
  // arrays below 1 MiB share allocations of 4 MiB: a plan has some fifty of
  // them, and an allocation costs 1 to 10 us and its release as much again
  size_t bytes = (std::max<size_t>(n, 1) * sizeof(T) + 255) & ~(size_t)255;
  const bool small = bytes < kSlabShare;
  if (small && bytes <= pl->slab_cap - pl->slab_used) {
    *p = (T *)(pl->slab + pl->slab_used);
    pl->slab_used += bytes;
    return GSIS_OK;
  }
  const size_t used = bytes;
  if (small) bytes = kSlabBytes;
  hipError_t e = hipMalloc(&v, bytes);
  if (e != hipSuccess)
    return fail(pl->ctx, GSIS_E_OOM, "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
  pl->allocs.push_back(v);
  if (small) {
    pl->slab = (char *)v;
    pl->slab_used = used;
    pl->slab_cap = bytes;
  }
  *p = (T *)v;
  return GSIS_OK;
}

template <typename T>
gsis_status upload(gsis_plan *pl, T **p, const std::vector<T> &h) {
  gsis_status st = dalloc(pl, p, h.size());
  if (st) return st;
  if (!h.empty()) HIPCHK(pl->ctx, hipMemcpy(*p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice));
  return GSIS_OK;
}

// Small host arrays that go to the device in one copy.
struct Pack {
  std::vector<char> h;
  std::vector<std::pair<void **, size_t>> at;
  template <typename T>
  void add(T **p, const std::vector<T> &v) {
    at.push_back({(void **)p, h.size()});
    h.resize((h.size() + v.size() * sizeof(T) + 255) & ~(size_t)255);
    if (!v.empty()) memcpy(h.data() + at.back().second, v.data(), v.size() * sizeof(T));
  }
  gsis_status commit(gsis_plan *pl) {
    char *d = nullptr;
    gsis_status st = dalloc(pl, &d, h.size());
    if (st) return st;
    if (!h.empty()) HIPCHK(pl->ctx, hipMemcpy(d, h.data(), h.size(), hipMemcpyHostToDevice));
    for (auto &e : at) *e.first = d + e.second;
    return GSIS_OK;
  }
};

// P.S for the plan alone (descriptor upload, block counts).
gsis_status make_single_set(gsis_plan *pl);
// Frees the adjoint's host-side state (device memory goes with the plan).
void adjoint_release(gsis_plan *pl);
// gsis_plan_create for one of `share` plans that run together.
gsis_status plan_create_shared(gsis_ctx *ctx, const gsis_problem *p, const gsis_options *o,
                               int share, gsis_plan **out);
// gsis_plan_reset without the wait at its end.
gsis_status plan_reset_enqueue(gsis_plan *pl);
