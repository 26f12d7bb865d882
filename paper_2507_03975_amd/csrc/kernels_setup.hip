// kernels_setup.hip -- a plan's set-up and its restart and read-out on gfx950:
// checks of the problem's fields, the coefficients of every cell, the
// per-quadrant records, the level-0 synthetic operator and its Galerkin
// coarsening. All of it touches each cell a few times; on the host it was
// most of a one-shot solve (256 x 256 cells: 4.5 ms of 14.6, 1024 x 1024:
// 141 ms), with the fields copied to the host and the results back.
//
// The arithmetic is the same operations in the same order as a scalar
// evaluation without fused multiply-adds, so a plan's coefficients do not
// depend on which side formed them.
#include "gsis_internal.h"
#include "wave_ops.h"

#include <algorithm>

#pragma clang fp contract(off)

namespace gsis {
namespace {

constexpr int kSB = 256;
inline int nb_(long long n) { return (int)((n + kSB - 1) / kSB); }

// Kinds of a bad cell, in the order they are reported for one cell.
// bad[0]: smallest 8 * cell + kind; bad[1]: smallest index into bnd_in.
__global__ void k_check_cells(int N, const double *sa, const double *ss, const double *q,
                              const double *cv, const double *T0, double *st,
                              unsigned long long *bad) {
  const int c = blockIdx.x * kSB + threadIdx.x;
  if (c >= N) return;
  const double a = sa[c], s = ss[c], v = q[c];
  int kind = -1;
  if (!isfinite(a) || a < 0) kind = kBadSigA;
  else if (!isfinite(s) || s < 0) kind = kBadSigS;
  else if (!(a + s > 0)) kind = kBadSigT;
  else if (!isfinite(v)) kind = kBadQ;
  if (kind >= 0) atomicMin(&bad[0], 8ull * c + kind);
  if (cv) {
    kind = !(cv[c] > 0) || !isfinite(cv[c]) ? kBadCv : !(T0[c] >= 0) || !isfinite(T0[c]) ? kBadT0 : -1;
    if (kind >= 0) atomicMin(&bad[2], 8ull * c + kind);
  }
  st[c] = a + s;
}

// The caller's boundary intensities in the internal ordinate order.
__global__ void k_setup_bnd(long long n, int K, const double *src, const int *perm, double *dst,
                            unsigned long long *bad) {
  const long long t = blockIdx.x * (long long)kSB + threadIdx.x;
  if (t >= n) return;
  const long long f = t / K;
  const int kk = (int)(t - f * K);
  const long long o = f * K + perm[kk];
  const double v = src[o];
  if (!isfinite(v)) atomicMin(&bad[1], (unsigned long long)o);
  dst[t] = v;
}

// Per cell: the adaptive least-squares coefficients (Eqs. shifted_j,
// LSF_mdf), kappa on its wall faces (Eqs. macro_bc_delta_flux,
// macro_bc_delta_flux2) and its row of the level-0 synthetic operator times V
// (Eqs. MSE_d_mtx1, elem_mtx_M, Gamma_ij_com2).
__global__ void k_setup_cells(SetupArgs a) {
  const int c = blockIdx.x * kSB + threadIdx.x;
  const int nx = a.nx, ny = a.ny;
  if (c >= nx * ny) return;
  const int j = c / nx, i = c - j * nx;
  const double *st = a.st;
  const double dx = a.dx, dy = a.dy, sc = st[c];
  const bool hE = i + 1 < nx, hW = i > 0, hN = j + 1 < ny, hS = j > 0;
  const double sE = hE ? st[c + 1] : 0.0, sW = hW ? st[c - 1] : 0.0;
  const double sN = hN ? st[c + nx] : 0.0, sS = hS ? st[c - nx] : 0.0;
  // distance from x_c to the (shifted) neighbour point along the normal
  // (Eq. shifted_j): half a cell to the face, then sigma_nb/sigma_c times
  // the half cell beyond it; plain least squares uses the centre
  auto dist = [&](bool has, double snb, double h) {
    if (!has) return 0.0;
    return a.alsm ? 0.5 * h + (snb / sc) * (0.5 * h) : h;
  };
  const double dE = dist(hE, sE, dx), dW = dist(hW, sW, dx);
  const double dN = dist(hN, sN, dy), dS = dist(hS, sS, dy);
  const double mx = dE * dE + dW * dW, my = dN * dN + dS * dS;
  a.cE[c] = mx > 0 ? dE / mx : 0.0;
  a.cW[c] = mx > 0 ? dW / mx : 0.0;
  a.cN[c] = my > 0 ? dN / my : 0.0;
  a.cS[c] = my > 0 ? dS / my : 0.0;
  const double kx = 2.0 / (3.0 * sc * dx) + 0.25, ky = 2.0 / (3.0 * sc * dy) + 0.25;
  if (!hW) a.kappa[j] = kx;
  if (!hE) a.kappa[ny + j] = kx;
  if (!hS) a.kappa[2 * ny + i] = ky;
  if (!hN) a.kappa[2 * ny + nx + i] = ky;
  auto gx = [&](double s0, double s1) { return dy * 2.0 / (3.0 * (s0 * dx + s1 * dx)); };
  auto gy = [&](double s0, double s1) { return dx * 2.0 / (3.0 * (s0 * dy + s1 * dy)); };
  const double aE = hE ? gx(sc, sE) : 0.0, aN = hN ? gy(sc, sN) : 0.0;
  double d = a.V * a.sa[c];
  d += hE ? aE : dy * kx;
  d += hW ? gx(sW, sc) : dy * kx;
  d += hN ? aN : dx * ky;
  d += hS ? gy(sS, sc) : dx * ky;
  a.diag[c] = d + a.V * a.tdiag;   // 1/(c dt) of Eq. elem_mtx_M (td form)
  a.ax[c] = aE;
  a.ay[c] = aN;
}

// Per-quadrant records in each quadrant's mirrored frame (cE, cW, cN, cS,
// sigma_t, sigma_t + pseudo-time shift) and the plane of the last, over 16 x
// 16 tiles: read by rows, passed through LDS, written along the stored
// diagonals. The shift is that of the increment-solve diagonal (Eqs. cfl_pse,
// tau_pse, elem_main_shifted); |sigma_i r^L - sigma_j r^R| is
// (sigma_i h + sigma_j h) / 2 for the face-normal width h.
constexpr int kST = 16;
__global__ void __launch_bounds__(kSB) k_setup_records(SetupArgs a) {
  __shared__ double sm[6][kST * kST];
  const int nx = a.nx, ny = a.ny, N = nx * ny;
  const int tw = (nx + kST - 1) / kST;
  const int i0 = (int)(blockIdx.x % tw) * kST, j0 = (int)(blockIdx.x / tw) * kST;
  {
    const int l = threadIdx.x, i = i0 + l % kST, j = j0 + l / kST;
    if (i < nx && j < ny) {
      const int c = j * nx + i;
      const double *st = a.st;
      double sh = a.cfl_p > 0 ? 1.0 / (a.cfl_p * a.dref) : 0.0;
      if (a.beta > 0) {
        double m = 0.0;
        if (i > 0) m = fmax(m, 0.5 * (st[c] + st[c - 1]) * a.dx);
        if (i + 1 < nx) m = fmax(m, 0.5 * (st[c] + st[c + 1]) * a.dx);
        if (j > 0) m = fmax(m, 0.5 * (st[c] + st[c - nx]) * a.dy);
        if (j + 1 < ny) m = fmax(m, 0.5 * (st[c] + st[c + nx]) * a.dy);
        sh += m / (a.beta * a.dref);
      }
      sm[0][l] = a.cE[c]; sm[1][l] = a.cW[c]; sm[2][l] = a.cN[c]; sm[3][l] = a.cS[c];
      // the time-dependent form's 1/(c dt) joins sigma_t in the residual's
      // -sigma_t I term and in the increment solve's diagonal (Eqs.
      // RTE_d_res, elem_mtx)
      sm[4][l] = st[c] + a.tdiag;
      sm[5][l] = st[c] + a.tdiag + sh;
    }
  }
  __syncthreads();
  // the thread's cell of the square in anti-diagonal order
  const int t = threadIdx.x, n = kST * kST;
  const int e = t < n / 2 + kST / 2 ? dg_corner(t) : 2 * kST - 2 - dg_corner(n - 1 - t);
  const int before = e < kST ? e * (e + 1) / 2 : n - (2 * kST - 1 - e) * (2 * kST - e) / 2;
  const int w = (e < kST ? 0 : e - kST + 1) + (t - before), u = e - w;
  for (int q = 0; q < 4; ++q) {
    const int x = (q & 1) ? nx - i0 - kST + u : i0 + u, y = (q & 2) ? ny - j0 - kST + w : j0 + w;
    if (x < 0 || x >= nx || y < 0 || y >= ny) continue;
    const int l = ((q & 2) ? kST - 1 - w : w) * kST + ((q & 1) ? kST - 1 - u : u);
    const size_t o = (size_t)q * N + dg_row0(x + y, nx, ny) + y;
    double2 *r = reinterpret_cast<double2 *>(a.cellq + 6 * o);
    r[0] = (q & 1) ? make_double2(sm[1][l], sm[0][l]) : make_double2(sm[0][l], sm[1][l]);
    r[1] = (q & 2) ? make_double2(sm[3][l], sm[2][l]) : make_double2(sm[2][l], sm[3][l]);
    r[2] = make_double2(sm[4][l], sm[5][l]);
    a.sdq[o] = sm[5][l];
    if (a.sdq_f) a.sdq_f[o] = (float)sm[5][l];
  }
}

// Sums of log ax and log ay over a level's interior faces, one pair per
// block (the mean couplings decide the aggregates).
__global__ void __launch_bounds__(kSB) k_log_sums(int nx, int ny, const double *ax,
                                                  const double *ay, double *part) {
  __shared__ double sh[2][kSB / 64];
  double x = 0.0, y = 0.0;
  const int n = nx * ny;
  for (int c = blockIdx.x * kSB + threadIdx.x; c < n; c += gridDim.x * kSB) {
    const int j = c / nx, i = c - j * nx;
    if (i + 1 < nx) x += log(ax[c]);
    if (j + 1 < ny) y += log(ay[c]);
  }
  x = wave_sum64(x);
  y = wave_sum64(y);
  if ((threadIdx.x & 63) == 0) { sh[0][threadIdx.x >> 6] = x; sh[1][threadIdx.x >> 6] = y; }
  __syncthreads();
  if (threadIdx.x < 2) {
    const double *s = sh[threadIdx.x];
    part[2 * blockIdx.x + threadIdx.x] = ((s[0] + s[1]) + s[2]) + s[3];
  }
}

// Galerkin coarsening by fx x fy aggregates: one thread per coarse cell, its
// children row by row.
__global__ void k_coarsen(int nx, int ny, int fx, int fy, const double *dg, const double *ax,
                          const double *ay, int cnx, int cny, double *cdg, double *cax,
                          double *cay) {
  const int C = blockIdx.x * kSB + threadIdx.x;
  if (C >= cnx * cny) return;
  const int J = C / cnx, I = C - J * cnx;
  double d = 0.0, x = 0.0, y = 0.0;
  for (int dj = 0; dj < fy; ++dj)
    for (int di = 0; di < fx; ++di) {
      const int i = fx * I + di, j = fy * J + dj;
      if (i >= nx || j >= ny) continue;
      const int c = j * nx + i;
      d += dg[c];
      if (i + 1 < nx) {
        if (di + 1 < fx) d -= 2.0 * ax[c];
        else x += ax[c];
      }
      if (j + 1 < ny) {
        if (dj + 1 < fy) d -= 2.0 * ay[c];
        else y += ay[c];
      }
    }
  cdg[C] = d;
  cax[C] = x;
  cay[C] = y;
}

// The iterate's start (all but the intensities): phi and T of the warm start,
// no pending correction, empty histories, counters and flags cleared, the
// hand-over buffer empty.
__global__ void k_plan_reset(ResetArgs a) {
  const size_t t = blockIdx.x * (size_t)kSB + threadIdx.x;
  if (t < (size_t)a.N) {
    const double p = a.phi0 ? a.phi0[t] : 0.0;
    a.phi[t] = p;
    a.delta[t] = 0.0;
    if (a.base) a.base[t] = p;     // FP32-mixed: I^0 = Itilde + phi0/(4 pi)
    if (a.T0) a.Tm[t] = a.T0[t];
  }
  if (t < (size_t)a.max_iter) { a.err_hist[t] = 0.0; a.tres_hist[t] = 0.0; }
  if (t < a.n_tres) a.tres_part[t] = 0.0;
  if (t < a.n_hand) a.hand[t] = kHandEmpty;
  if (t < kStateWords) a.state[t] = 0;
  if (t == 0) {
    *a.vcycles = 0.0;
    // Err of the last iteration and the smallest ||phi^{m+1} - phi^m||_V so
    // far (divergence test)
    a.last_err[0] = 0.0;
    a.last_err[1] = INFINITY;
  }
}

// phi, F and the histories of the current iterate: F = F_half plus the
// pending correction's flux, delta/(4 pi) sum_k w Omega_k. Nothing if the
// recurrence's workgroups lost each other (state[4]); a NULL output is skipped.
__global__ void k_plan_read(ReadArgs a) {
  const int t = blockIdx.x * kSB + threadIdx.x;
  if (a.state[4] != 0) return;
  if (t < a.N) {
    const double d = a.delta[t] / kFourPi;
    if (a.ophi) a.ophi[t] = a.phi[t];
    a.oFx[t] = __builtin_fma(d, a.swm, a.Fx[t]);
    a.oFy[t] = __builtin_fma(d, a.swe, a.Fy[t]);
  }
  if (t < a.state[0]) {
    if (a.oerr) a.oerr[t] = a.err_hist[t];
    if (a.otres) a.otres[t] = a.tres_hist[t];
  }
}

}  // namespace

void launch_check_cells(int N, const double *sa, const double *ss, const double *q,
                        const double *cv, const double *T0, double *st, unsigned long long *bad,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_check_cells, dim3(nb_(N)), dim3(kSB), 0, s, N, sa, ss, q, cv, T0, st, bad);
}
void launch_setup_bnd(long long n, int K, const double *src, const int *perm, double *dst,
                      unsigned long long *bad, hipStream_t s) {
  hipLaunchKernelGGL(k_setup_bnd, dim3(nb_(n)), dim3(kSB), 0, s, n, K, src, perm, dst, bad);
}
void launch_setup_cells(const SetupArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_setup_cells, dim3(nb_((long long)a.nx * a.ny)), dim3(kSB), 0, s, a);
  const int nt = ((a.nx + kST - 1) / kST) * ((a.ny + kST - 1) / kST);
  hipLaunchKernelGGL(k_setup_records, dim3(nt), dim3(kSB), 0, s, a);
}
int launch_log_sums(const MGLevel &L, double *part, hipStream_t s) {
  const int nb = std::min(nb_((long long)L.nx * L.ny), kLogBlocks);
  hipLaunchKernelGGL(k_log_sums, dim3(nb), dim3(kSB), 0, s, L.nx, L.ny, L.ax, L.ay, part);
  return nb;
}
void launch_coarsen(const MGLevel &F, const MGLevel &C, hipStream_t s) {
  hipLaunchKernelGGL(k_coarsen, dim3(nb_((long long)C.nx * C.ny)), dim3(kSB), 0, s, F.nx, F.ny,
                     F.fx, F.fy, F.diag, F.ax, F.ay, C.nx, C.ny, C.diag, C.ax, C.ay);
}
void launch_plan_reset(const PlanDev &P, size_t n_tres, hipStream_t s) {
  ResetArgs a;
  a.N = P.N;
  a.max_iter = P.max_iter;
  a.n_tres = n_tres;
  a.n_hand = hand_parts(P) > 1 ? (size_t)P.K * (hand_parts(P) - 1) * P.nx : 0;
  a.phi0 = P.phi0; a.T0 = P.T0;
  a.phi = P.phi; a.delta = P.delta;
  a.base = P.precision == GSIS_FP32_MIXED ? P.base : nullptr;
  a.Tm = P.Tm;
  a.err_hist = P.err_hist; a.tres_hist = P.tres_hist; a.tres_part = P.tres_part;
  a.vcycles = synth_vcycle_total(P);
  a.last_err = P.last_err;
  a.hand = P.hand;
  a.state = P.state;
  const size_t n = std::max({(size_t)a.N, (size_t)a.max_iter, a.n_tres, a.n_hand, (size_t)8});
  hipLaunchKernelGGL(k_plan_reset, dim3((unsigned)((n + kSB - 1) / kSB)), dim3(kSB), 0, s, a);
}
void launch_plan_read(const PlanDev &P, double swm, double swe, double *phi, double *Fx, double *Fy,
                      double *err, double *tres, hipStream_t s) {
  ReadArgs a{P.N, P.state, P.phi, P.Fx, P.Fy, P.delta, P.err_hist, P.tres_hist,
             swm, swe, phi, Fx, Fy, err, tres};
  const int n = err || tres ? std::max(P.N, P.max_iter) : P.N;
  hipLaunchKernelGGL(k_plan_read, dim3(nb_(n)), dim3(kSB), 0, s, a);
}

}  // namespace gsis
