// kernels_synth.hip -- macroscopic (synthetic) step of GSIS on gfx950.
//
//  hot     : HoT_c = F_c + grad(phi)_c / (3 sigma_t) with the adaptive
//            least-squares gradient (Eqs. GSIS_HoT, LSF_mdf); right-hand side
//            b_c = V q - sum_int A 1/2 (HoT_c + HoT_nb).n
//                  - sum_bnd A (F_T.n - kappa phi_half)        (Eqs. MSE_d, Fij_d,
//                                                  macro_bc_delta_flux),
//            formed by the kernel that starts the CG
//  solve   : D1 phi' = b, D1 = V sigma_a + sum_int A Gamma (.) + sum_bnd A kappa
//            (Eqs. Gamma_ij_def, MSE_d_mtx1, elem_mtx_M, Gamma_ij_com2), by
//            CG (one reduction per iteration, the Chronopoulos-Gear form)
//            preconditioned with a geometric multigrid V-cycle (2x2
//            aggregation, Galerkin coarse operators, red-black Gauss-Seidel
//            smoothing, dense inverse on the coarsest level).
//  update  : delta = phi' - phi_half (Eq. GSIS_update, applied lazily by the
//            transport kernels), Err (Eq. Err_W), next source.
//
// Every kernel takes its problem from a SynthDesc record. A launch covers one
// problem (block table NULL) or many: the table maps each block to (problem,
// block of that problem), so the problems of a batch advance together while
// each keeps its own CG scalars, multigrid hierarchy and stop flags.
// All reductions are two-stage with a fixed order, so results repeat bit for
// bit, and a problem gets the same phi and F alone or in a batch (a small one's
// solve is one kernel alone and several beside larger problems, with the same
// sums in the same order).
#include "gsis_internal.h"
#include "wave_ops.h"

#include <algorithm>
#include <cstring>
#include <type_traits>

namespace gsis {
namespace {

constexpr int kRedBlock = 256;

// v of the lane given by DPP control C (a permutation within rows of 16)
template <int C>
__device__ inline double dpp_d(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, C, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), C, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ inline double read_lane(double v, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Sum over a full wave in a fixed order: quads by the lane permutations
// xor 1 and xor 2 (every lane of a quad ends with the same sum, as addition
// commutes exactly), the four quads of a row by rotations of 4 and 8, then
// the four rows' sums read as scalars and added pairwise.
__device__ inline double wave_sum(double v) {
  v += dpp_d<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_d<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_d<0x124>(v);   // row_ror:4
  v += dpp_d<0x128>(v);   // row_ror:8
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Sum over the block (every lane of it active, blockDim a multiple of 64):
// wave sums, then the waves' sums in wave order. Every thread gets the same
// value; sh needs one entry per wave.
__device__ inline double block_sum(double v, double *sh) {
  const double w = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = w;
  __syncthreads();
  double r = 0.0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += sh[k];
  __syncthreads();
  return r;
}

// the same for two values; sh needs two entries per wave
__device__ inline void block_sum2(double &u, double &v, double *sh) {
  const double a = wave_sum(u), b = wave_sum(v);
  if ((threadIdx.x & 63) == 0) {
    sh[2 * (threadIdx.x >> 6)] = a;
    sh[2 * (threadIdx.x >> 6) + 1] = b;
  }
  __syncthreads();
  u = v = 0.0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) { u += sh[2 * k]; v += sh[2 * k + 1]; }
  __syncthreads();
}

// (i, j) of cell c on a grid nx wide without an integer division: the
// quotient from the hardware reciprocal is off by at most one for c < 2^28
// and is corrected.
__device__ inline void cell_ij(int c, int nx, int &i, int &j) {
  int q = (int)((double)c * __builtin_amdgcn_rcp((double)nx));
  int r = c - q * nx;
  if (r < 0) { --q; r += nx; } else if (r >= nx) { ++q; r -= nx; }
  i = r; j = q;
}

// Problem descriptors and block tables are read through the constant
// address space: they do not change while a kernel runs, so their
// (wave-uniform) fields become scalar loads served by the scalar cache
// rather than vector loads, each of which would cost a memory round trip.
typedef __attribute__((address_space(4))) const SynthDesc CDesc;
__device__ inline CDesc &cdesc(const SynthDesc *ds, int p) { return ((CDesc *)ds)[p]; }
// a level's record copied out of a descriptor field by field
__device__ inline LevelDev level(CDesc &D, int l) {
  __attribute__((address_space(4))) const LevelDev &s = D.lev[l];
  LevelDev L;
  L.nx = s.nx; L.ny = s.ny; L.fx = s.fx; L.fy = s.fy;
  L.dg = s.dg; L.ax = s.ax; L.ay = s.ay; L.x = s.x; L.b = s.b; L.xs = s.xs;
  return L;
}

// The block's problem and its block index within that problem.
struct Blk { int p, lb; };
__device__ inline Blk blk(const int2 *bt) {
  if (!bt) return {0, (int)blockIdx.x};
  const __attribute__((address_space(4))) int *q = (const __attribute__((address_space(4))) int *)bt;
  return {q[2 * blockIdx.x], q[2 * blockIdx.x + 1]};
}

// ---------------------------------------------------------------- HoT / RHS
// COMBINE: phi and F of I^{m+1/2} are first summed from the four quadrant
// partials (for the cell and, phi only, its neighbours; quadrants in order,
// plus the FP32-mixed base term), and the cell's values stored.
template <bool COMBINE>
__global__ void k_hot(const SynthDesc *ds, const int2 *bt) {
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1];   // tested after the operands are loaded
  const int nx = D.nx, ny = D.ny, N = D.N;
  const int c = B.lb * kRedBlock + threadIdx.x;
  if (c >= N) return;
  int i, j;
  cell_ij(c, nx, i, j);
  const int ce = i + 1 < nx ? c + 1 : c, cw = i > 0 ? c - 1 : c;
  const int cn = j + 1 < ny ? c + nx : c, cs = j > 0 ? c - nx : c;
  double u, ue, uw, un, us, fx, fy;
  if (COMBINE) {
    const double *P = D.mom_part;
    auto phi_at = [&](int cc) {
      double s0 = 0.0;
      for (int q = 0; q < 4; ++q) s0 += P[(size_t)(3 * q) * N + cc];
      if (D.fp32) s0 += D.phi[cc] / kFourPi * D.sw;
      return s0;
    };
    u = phi_at(c); ue = phi_at(ce); uw = phi_at(cw); un = phi_at(cn); us = phi_at(cs);
    double sx = 0.0, sy = 0.0;
    for (int q = 0; q < 4; ++q) {
      sx += P[(size_t)(3 * q + 1) * N + c];
      sy += P[(size_t)(3 * q + 2) * N + c];
    }
    if (D.fp32) {
      const double sub = D.phi[c] / kFourPi;
      sx += sub * D.swm;
      sy += sub * D.swe;
    }
    fx = sx; fy = sy;
  } else {
    const double *phih = D.phih;
    u = phih[c]; ue = phih[ce]; uw = phih[cw]; un = phih[cn]; us = phih[cs];
    fx = D.Fx[c]; fy = D.Fy[c];
  }
  double hx, hy;
  if (D.hot_face) {
    // transport face fluxes on the cell's east and north faces (sums of the
    // four quadrant partials, in order) minus the compact diffusion flux
    // Gamma_f (phi_c - phi_nb); A Gamma_f is the operator's off-diagonal
    const double *FT = D.ftp;
    double tx = 0.0, ty = 0.0;
    for (int q = 0; q < 4; ++q) {
      tx += FT[(size_t)(2 * q) * N + c];
      ty += FT[(size_t)(2 * q + 1) * N + c];
    }
    const double gE = D.lev[0].ax[c] / D.dy, gN = D.lev[0].ay[c] / D.dx;
    hx = i + 1 < nx ? tx - gE * (u - ue) : 0.0;
    hy = j + 1 < ny ? ty - gN * (u - un) : 0.0;
  } else {
    const double gx = D.cE[c] * (ue - u) - D.cW[c] * (uw - u);
    const double gy = D.cN[c] * (un - u) - D.cS[c] * (us - u);
    hx = fx + gx / (3.0 * D.sig_t[c]);
    hy = fy + gy / (3.0 * D.sig_t[c]);
  }
  if (f1 != 0) return;
  if (COMBINE) {
    D.phih[c] = u;
    D.Fx[c] = fx;
    D.Fy[c] = fy;
  }
  D.hx[c] = hx;
  D.hy[c] = hy;
}

// The time-dependent form's material temperature of sub-iteration sub: T^m,
// then the sub-iterates in two alternating buffers.
__device__ inline double *t_sub(CDesc &D, int sub) {
  return sub == 0 ? D.Tm : ((sub - 1) & 1) ? D.Tsub1 : D.Tsub0;
}

// b_c of cell c = (i, j) from the HoT of the cell and its neighbours (central
// faces), or from the face values h of its faces (transport faces: hx[c] on
// the cell's east face, hy[c] on its north face, normals +x, +y). The
// time-dependent form adds V (rho^n / (c dt) + sigma_a a c T^4) with T the
// temperature Ts of the sub-iteration (D1 carries V / (c dt) on its diagonal):
// then D1 rho' = b is D1 d_rho = R1 of Eqs. MSE_d1, R1_def at rho' = rho + d_rho.
__device__ inline double rhs_at(CDesc &D, int c, int i, int j, const double *Ts) {
  const int nx = D.nx, ny = D.ny;
  const double dx = D.dx, dy = D.dy;
  const double *hx = D.hx, *hy = D.hy, *bflux = D.bflux, *kappa = D.kappa;
  const double ph = D.phih[c];
  const bool tf = D.hot_face != 0;
  double s = dx * dy * D.q[c];
  if (D.td) {
    const double T = Ts[c], T2 = T * T;
    s += dx * dy * (D.rho_n[c] * D.tdiag + D.sig_a[c] * (D.ca * (T2 * T2)));
  }
  // east / west (area dy), north / south (area dx)
  if (i + 1 < nx) s -= dy * (tf ? hx[c] : 0.5 * (hx[c] + hx[c + 1]));
  else s -= dy * (bflux[ny + j] - kappa[ny + j] * ph);
  if (i > 0) s += dy * (tf ? hx[c - 1] : 0.5 * (hx[c] + hx[c - 1]));
  else s -= dy * (bflux[j] - kappa[j] * ph);
  if (j + 1 < ny) s -= dx * (tf ? hy[c] : 0.5 * (hy[c] + hy[c + nx]));
  else s -= dx * (bflux[2 * ny + nx + i] - kappa[2 * ny + nx + i] * ph);
  if (j > 0) s += dx * (tf ? hy[c - nx] : 0.5 * (hy[c] + hy[c - nx]));
  else s -= dx * (bflux[2 * ny + i] - kappa[2 * ny + i] * ph);
  return s;
}

// Scalar slots. r.z of CG iteration k sits in slot rz_slot(k) (two
// alternating slots, so a kernel can read iteration k-1's value while its
// block 0 stores iteration k's).
enum { S_RZ = 0, S_ZW = 1, S_RR = 2, S_BB = 3, S_ALPHA = 4, S_BETA = 5, S_STOP = 6,
       S_NIT = 7, S_RZ1 = 8, S_ALPHA1 = 9, S_VCYCLES = 10 };
__host__ __device__ inline int rz_slot(int k) { return (k & 1) ? S_RZ1 : S_RZ; }
__host__ __device__ inline int alpha_slot(int k) { return (k & 1) ? S_ALPHA1 : S_ALPHA; }

// r of V-cycle v (v = 0 after the warm start, v = it + 1 after CG iteration
// it): the buffers alternate, so a kernel that forms r_{v} for its tile and
// halo never overwrites the r_{v-1} that neighbouring tiles still read.
__device__ inline double *cg_rv(CDesc &D, int v) { return (v & 1) ? D.cg_r2 : D.cg_r; }

// CG kernels run unless the outer iteration is done (state[1]) or this
// synthetic solve has converged (state[3]).
__device__ inline bool cg_off(const int32_t *st) { return st[1] != 0 || st[3] != 0; }

inline int nblk(int n) { return (n + kRedBlock - 1) / kRedBlock; }
__host__ __device__ inline int nblk_d(int n) { return (n + kRedBlock - 1) / kRedBlock; }

// Block partials of a problem's reductions, in separate regions of its red
// array (nb = level-0 blocks of 256 cells): [0, nb) r.r, [nb, 2 nb) b.b,
// then three regions of ntp = max(nb, level-0 tiles) slots: r.z (one per
// level-0 tile, or per block of cells when the whole V-cycle ran in one
// workgroup), r.r once more, one per level-0 tile, from the tile kernel
// that makes the CG update, and z.Az (like r.z). A reduction is finished by the
// kernel that needs its value: every block of it sums the partials in the
// same fixed order, so all blocks hold the same number and results repeat
// bit for bit; block 0 stores it for later kernels. This saves a launch
// per reduction (folding the finish into the producing kernel instead would
// need a device-scope release per block, which on a GPU whose XCDs each
// have their own L2 writes back the L2 every time).
__device__ inline double *red_rr(CDesc &D) { return D.red; }
__device__ inline double *red_bb(CDesc &D) { return D.red + nblk_d(D.N); }
__device__ inline double *red_rz(CDesc &D) { return D.red + 2 * nblk_d(D.N); }
__device__ inline double *red_rrt(CDesc &D) { return D.red + 2 * nblk_d(D.N) + D.ntp; }
__device__ inline double *red_zw(CDesc &D) { return D.red + 2 * nblk_d(D.N) + 2 * D.ntp; }
__device__ inline int n_rz(CDesc &D) { return D.lc == 0 ? nblk_d(D.N) : D.ntile0; }

// The thread's first partial, loaded early (before a kernel waits for its
// flags), and the sum of all n partials: thread t adds p[t], p[t + blockDim],
// ... in that order, then block_sum.
__device__ inline double first_partial(const double *p, int n) {
  return p[(int)threadIdx.x < n ? threadIdx.x : 0];   // sum_partials drops what is past n
}
__device__ inline double thread_partials(const double *p, int n, double first) {
  double v = (int)threadIdx.x < n ? first : 0.0;
  // sixteen loads in flight at a time, added in order (terms past n add 0)
  constexpr int U = 16;
  for (int t0 = threadIdx.x + blockDim.x; t0 < n; t0 += U * (int)blockDim.x) {
    double w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * (int)blockDim.x;
      w[u] = t < n ? p[t] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v += w[u];
  }
  return v;
}
__device__ inline double sum_partials(const double *p, int n, double *sh, double first) {
  return block_sum(thread_partials(p, n, first), sh);
}

// r.r of the iterate just updated (partials per level-0 tile when the tile
// kernel made the update, else per block of cells): iteration count and
// convergence test against STOP; first (after the warm start): also b.b,
// the count reset and STOP = max(rtol^2 r0.r0, 1e-28 b.b). Every thread of
// the block returns the same decision; thread 0 stores the scalars and the
// flag. Its operands can be loaded early (rr_prefetch), before the caller
// waits for its flags.
struct RRTest {
  const double *rr, *bb;       // partials
  int nrr, nb;
  bool first;
  double *scal;
  int32_t *state;
  double rtol;
};
struct RRPre {
  double rr, bb, stop;
};
__device__ inline RRTest rr_test(CDesc &D, bool first, bool tiles) {
  RRTest T;
  T.nb = nblk_d(D.N);
  T.rr = tiles ? red_rrt(D) : red_rr(D);
  T.nrr = tiles ? D.ntile0 : T.nb;
  T.bb = red_bb(D);
  T.first = first;
  T.scal = D.scal;
  T.state = D.state;
  T.rtol = D.rtol;
  return T;
}
__device__ inline RRPre rr_prefetch(const RRTest &T) {
  RRPre q;
  q.rr = first_partial(T.rr, T.nrr);
  q.bb = T.first ? first_partial(T.bb, T.nb) : 0.0;
  q.stop = T.scal[S_STOP];
  return q;
}
__device__ inline RRPre rr_prefetch(CDesc &D, bool first, bool tiles) {
  return rr_prefetch(rr_test(D, first, tiles));
}
__device__ inline bool finish_rr(const RRTest &T, double *sh, const RRPre &q) {
  const double rr = sum_partials(T.rr, T.nrr, sh, q.rr);
  double stop = q.stop, bb = 0.0;
  if (T.first) {
    bb = sum_partials(T.bb, T.nb, sh, q.bb);
    stop = fmax(T.rtol * T.rtol * rr, 1e-28 * bb);
  }
  const bool conv = !(rr > stop);
  if (threadIdx.x == 0) {
    double *scal = T.scal;
    scal[S_RR] = rr;
    if (T.first) {
      scal[S_BB] = bb;
      scal[S_STOP] = stop;
    }
    const double nit = T.first ? 0.0 : scal[S_NIT] + 1.0;
    scal[S_NIT] = nit;
    // converged: 1 + the CG iterations it took (the host's next check point)
    if (conv) T.state[3] = 1 + (int32_t)nit;
  }
  return conv;
}
__device__ inline bool finish_rr(CDesc &D, bool first, bool tiles, double *sh, const RRPre &q) {
  return finish_rr(rr_test(D, first, tiles), sh, q);
}

// The r.r test of the last CG iteration when the iteration cap ends the
// solve (one workgroup per problem).
__global__ void k_finish_rr(const SynthDesc *ds) {
  __shared__ double sh[kRedBlock];
  CDesc &D = cdesc(ds, blockIdx.x);
  const RRPre q = rr_prefetch(D, false, false);
  if (cg_off(D.state)) return;
  (void)finish_rr(D, false, false, sh, q);
}

// The r.r test of CG iteration v - 1 (v > 0) on its level-0 tile partials,
// for a problem whose V-cycle starts with a tile level: the test the level-1
// kernel of V-cycle v would make, run on its own when the host is about to
// look at the flags (that V-cycle's later kernels, which the test would
// usually turn into no-ops, are then launched only if it fails).
__global__ void k_rr_test(const SynthDesc *ds) {
  __shared__ double sh[kRedBlock];
  CDesc &D = cdesc(ds, blockIdx.x);
  const RRPre q = rr_prefetch(D, false, true);
  if (cg_off(D.state)) return;
  (void)finish_rr(D, false, true, sh, q);
}

// Start of a synthetic solve: warm start x = phi, clear the converged flag;
// r = b - A x; partials of r.r and b.b.
// RHS: the right-hand side b is formed here from the HoT (and stored)
// rather than read.
// MODE 0: b given in rhs (the adjoint), warm start phi; 1: b from the HoT
// (rhs_at), warm start phi; 3: as 1 with the level-0 iterate as warm start
// (the time-dependent form's later sub-iterations); 2: the face-averaged
// balance (Eq. Fij_d) by a
// defect-correction sub-iteration: b = rhs_at + corr(x) with x the level-0
// iterate, which is also the warm start, and corr_c = sum over interior
// faces of a_f (x_c - x_nb) + A_f (w_c + w_nb) . n_f / 2, a_f = A_f Gamma_f
// the operator's off-diagonals and w = grad(x) / (3 sigma_t) from
// k_wide_grad: then D1 x' = b is D1 (x' - x) = R1(x).
template <int MODE>
__global__ void k_cg_begin(const SynthDesc *ds, const int2 *bt, int sub) {
  __shared__ double sh[kRedBlock];
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1];   // tested after the operands are loaded
  const int c = B.lb * kRedBlock + threadIdx.x;
  const LevelDev L = level(D, 0);
  const bool in = c < D.N;
  const int cc = in ? c : 0;
  int i, j;
  cell_ij(cc, L.nx, i, j);
  const bool hE = i + 1 < L.nx, hW = i > 0, hN = j + 1 < L.ny, hS = j > 0;
  // warm start x for the cell and its neighbours (this kernel writes x)
  const double *X = MODE >= 2 ? L.x : D.phi;
  const double xc = X[cc], xe = X[hE ? cc + 1 : cc], xw = X[hW ? cc - 1 : cc];
  const double xn = X[hN ? cc + L.nx : cc], xs = X[hS ? cc - L.nx : cc];
  const double dg = L.dg[cc], aE = L.ax[cc], aW = L.ax[hW ? cc - 1 : cc];
  const double aN = L.ay[cc], aS = L.ay[hS ? cc - L.nx : cc];
  double b = MODE != 0 ? rhs_at(D, cc, i, j, D.td ? t_sub(D, sub) : nullptr) : D.rhs[cc];
  if (MODE == 2) {
    const double *WX = D.wx, *WY = D.wy;
    const double wxc = WX[cc], wyc = WY[cc];
    const double hdy = 0.5 * D.dy, hdx = 0.5 * D.dx;
    double corr = 0.0;
    if (hE) corr += aE * (xc - xe) + hdy * (wxc + WX[cc + 1]);
    if (hW) corr += aW * (xc - xw) - hdy * (wxc + WX[cc - 1]);
    if (hN) corr += aN * (xc - xn) + hdx * (wyc + WY[cc + L.nx]);
    if (hS) corr += aS * (xc - xs) - hdx * (wyc + WY[cc - L.nx]);
    b += corr;
  }
  if (f1 != 0) return;
  double rr = 0.0, bb = 0.0;
  if (in) {
    double y = dg * xc;
    if (hE) y -= aE * xe;
    if (hW) y -= aW * xw;
    if (hN) y -= aN * xn;
    if (hS) y -= aS * xs;
    const double rc = b - y;
    if (MODE != 0) D.rhs[c] = b;
    L.x[c] = xc;
    D.cg_r[c] = rc;
    rr = rc * rc;
    bb = b * b;
  }
  if (B.lb == 0 && threadIdx.x == 0) D.state[3] = 0;
  double t = block_sum(rr, sh);
  if (threadIdx.x == 0) red_rr(D)[B.lb] = t;
  t = block_sum(bb, sh);
  if (threadIdx.x == 0) red_bb(D)[B.lb] = t;
}

// w = grad(x) / (3 sigma_t) of the level-0 iterate (the HoT's gradient
// coefficients), for the face-averaged balance; FIRST: x = phi^{m+1/2},
// also copied into the iterate (the sub-iterations start there).
template <bool FIRST>
__global__ void k_wide_grad(const SynthDesc *ds, const int2 *bt) {
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1];   // tested after the operands are loaded
  const int nx = D.nx, ny = D.ny;
  const int c = B.lb * kRedBlock + threadIdx.x;
  if (c >= D.N) return;
  int i, j;
  cell_ij(c, nx, i, j);
  const LevelDev L = level(D, 0);
  const double *X = FIRST ? D.phih : L.x;
  const double u = X[c];
  const double ue = i + 1 < nx ? X[c + 1] : u, uw = i > 0 ? X[c - 1] : u;
  const double un = j + 1 < ny ? X[c + nx] : u, us = j > 0 ? X[c - nx] : u;
  const double gx = D.cE[c] * (ue - u) - D.cW[c] * (uw - u);
  const double gy = D.cN[c] * (un - u) - D.cS[c] * (us - u);
  const double s3 = 3.0 * D.sig_t[c];
  if (f1 != 0) return;
  D.wx[c] = gx / s3;
  D.wy[c] = gy / s3;
  if (FIRST) L.x[c] = u;
}

// CG in the form of Chronopoulos and Gear: the V-cycle of iteration it
// gives z = M r and, on its finest level, w = A z with partials of
// gamma = r.z and delta = z.w in one pass, so an iteration needs a single
// global reduction. Then
//   beta = gamma / gamma_prev (0 on the first iteration),
//   alpha = gamma / (delta - beta gamma / alpha_prev) (gamma / delta first),
//   p = z + beta p, s = w + beta s (= A p), x += alpha p, r -= alpha s,
// which is preconditioned CG with A p carried by a recurrence instead of a
// product. s alternates between two buffers with the parity of it.
struct CGCoef {
  double be, al;
};
__device__ inline CGCoef cg_coef(bool first, double ga, double de, double ga_prev,
                                 double al_prev) {
  if (first) return {0.0, ga / de};
  const double be = ga / ga_prev;
  return {be, ga / (de - be * ga / al_prev)};
}
__device__ inline double *cg_s(CDesc &D, int it) { return (it & 1) ? D.cg_s1 : D.cg_s0; }
// the update's scalar operands, loaded before the caller waits for its flags
// (coef_sep: the coefficients themselves, from k_cg_coef)
struct UpdPre {
  double rz0, zw0, ga_prev, al_prev;
};
__device__ inline UpdPre upd_prefetch(CDesc &D, int it) {
  UpdPre q;
  if (D.coef_sep) {
    q.rz0 = it > 0 ? D.scal[S_BETA] : 0.0;
    q.zw0 = D.scal[alpha_slot(it)];
    q.ga_prev = q.al_prev = 0.0;
    return q;
  }
  q.rz0 = first_partial(red_rz(D), n_rz(D));
  q.zw0 = first_partial(red_zw(D), n_rz(D));
  q.ga_prev = it > 0 ? D.scal[rz_slot(it - 1)] : 1.0;
  q.al_prev = it > 0 ? D.scal[alpha_slot(it - 1)] : 1.0;
  return q;
}
// every block forms the coefficients from the same partials in the same
// order; block 0 stores gamma, delta, alpha and beta. With many partials
// (coef_sep) one workgroup does this in k_cg_coef instead, in the same
// order, and the blocks take the stored beta and alpha.
__device__ inline CGCoef upd_coef(CDesc &D, const Blk &B, int it, const UpdPre &q, double *sh) {
  if (D.coef_sep) return {q.rz0, q.zw0};
  double ga = thread_partials(red_rz(D), n_rz(D), q.rz0);
  double de = thread_partials(red_zw(D), n_rz(D), q.zw0);
  block_sum2(ga, de, sh);
  const CGCoef k = cg_coef(it == 0, ga, de, q.ga_prev, q.al_prev);
  if (B.lb == 0 && threadIdx.x == 0) {
    D.scal[rz_slot(it)] = ga;
    D.scal[alpha_slot(it)] = k.al;
    D.scal[S_BETA] = k.be;
    D.scal[S_ZW] = de;
  }
  return k;
}

// CG coefficients of iteration it for the problems whose level-0 tiles are
// many (coef_sep): one workgroup per problem sums the r.z and z.w partials
// (the order of upd_coef) and stores gamma, delta, alpha and beta, so each
// block of the update reads two scalars instead of every partial. Launched
// after V-cycle it.
constexpr int kCoefSepTiles = 2048;
__global__ void __launch_bounds__(kRedBlock) k_cg_coef(const SynthDesc *ds, int it) {
  __shared__ double sh[kRedBlock];
  CDesc &D = cdesc(ds, blockIdx.x);
  if (D.coef_sep != kCoefKernel) return;
  UpdPre q;
  q.rz0 = first_partial(red_rz(D), n_rz(D));
  q.zw0 = first_partial(red_zw(D), n_rz(D));
  q.ga_prev = it > 0 ? D.scal[rz_slot(it - 1)] : 1.0;
  q.al_prev = it > 0 ? D.scal[alpha_slot(it - 1)] : 1.0;
  if (cg_off(D.state)) return;
  double ga = thread_partials(red_rz(D), n_rz(D), q.rz0);
  double de = thread_partials(red_zw(D), n_rz(D), q.zw0);
  block_sum2(ga, de, sh);
  const CGCoef k = cg_coef(it == 0, ga, de, q.ga_prev, q.al_prev);
  if (threadIdx.x == 0) {
    D.scal[rz_slot(it)] = ga;
    D.scal[alpha_slot(it)] = k.al;
    D.scal[S_BETA] = k.be;
    D.scal[S_ZW] = de;
  }
}

// CG iteration it on every cell of a problem, with the partial of r.r.
// With all = 0 only problems whose whole V-cycle runs in the one-workgroup
// kernel take part: for the others the level-0 tile kernel of the next
// V-cycle makes the update.
__global__ void k_cg_update(const SynthDesc *ds, const int2 *bt, int it, int all) {
  __shared__ double sh[kRedBlock];
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  if (!all && D.lc > 0) return;
  const int32_t f1 = D.state[1], f3 = D.state[3];
  const int c = B.lb * kRedBlock + threadIdx.x;
  double *x = D.lev[0].x;
  const bool in = c < D.N;
  const int cc = in ? c : 0;
  const double zc = D.cg_z[cc], wc = D.cg_w[cc], xc = x[cc], rc0 = cg_rv(D, it)[cc];
  const double pc0 = it > 0 ? D.cg_p[cc] : 0.0, sc0 = it > 0 ? cg_s(D, it - 1)[cc] : 0.0;
  const UpdPre q = upd_prefetch(D, it);
  if (f1 != 0 || f3 != 0) return;
  const CGCoef k = upd_coef(D, B, it, q, sh);
  double v = 0.0;
  if (in) {
    const double pc = it > 0 ? fma(k.be, pc0, zc) : zc;
    const double sc = it > 0 ? fma(k.be, sc0, wc) : wc;
    D.cg_p[c] = pc;
    cg_s(D, it)[c] = sc;
    x[c] = fma(k.al, pc, xc);
    const double rc = fma(-k.al, sc, rc0);
    cg_rv(D, it + 1)[c] = rc;
    v = rc * rc;
  }
  double t = block_sum(v, sh);
  if (threadIdx.x == 0) red_rr(D)[B.lb] = t;
}

// ------------------------------------------------------------ multigrid
// Level l of a problem: vectors x, b are the CG's z, r on level 0 (r of
// V-cycle v).
__device__ inline double *lev_x(CDesc &D, int l) { return l == 0 ? D.cg_z : D.lev[l].x; }
__device__ inline const double *lev_b(CDesc &D, int l, int v) {
  return l == 0 ? cg_rv(D, v) : D.lev[l].b;
}

// Fine multigrid levels, one tile of kTW x kTH cells per workgroup (one
// thread per cell) with a ring of kHalo cells around it in LDS. Red-black
// Gauss-Seidel uses the colour (i + j) & 1 of the level (0 red, 1 black).
//
//  down: one V(1,1) pre-smoothing from x = 0 -- red x = b / d, then black
//        x = (b + sum a x_nb) / d -- then r = b - A x and the coarse
//        b = sum of r over each aggregate's fx x fy children. Starting from
//        zero makes every value a function of b, d and the couplings within
//        two cells, so the tile and its ring are computed without waiting
//        for other workgroups. The pre-smoothed x of the tile goes to the
//        level's spare vector xs, not to x. On level 0 after a CG step it
//        also makes that step's update: b = r_new =
//        r_old - alpha (w + beta s_old) is formed on the whole region from
//        r_old, w and s_old, which earlier kernels left complete.
//  up:   black x = (b + sum a (xs_nb + omega e_parent(nb))) / d with the
//        coarse correction e, then red x = (b + sum a x_nb) / d; the black
//        ring is recomputed so the red cells of the tile see final
//        neighbours. Level 0 has its own kernel (k_mg_up0). It
//        reads the pre-smoothed xs of the ring and writes the final x into a
//        different array, so tiles running later never see a neighbour's
//        final values in place of its pre-smoothed ones.
// Cells outside the level hold d = 1, b = 0 and no couplings.
constexpr int kTW = 32, kTH = 8, kHalo = 2;
constexpr int kRW = kTW + 2 * kHalo, kRH = kTH + 2 * kHalo, kRN = kRW * kRH;
static_assert(kTW * kTH == kRedBlock, "one thread per tile cell");

struct Tile {
  int nx, ny, i0, j0;
};
__device__ inline Tile tile_of(const LevelDev &L, int lb) {
  const int tx = (L.nx + kTW - 1) / kTW;
  int ti, tj;
  cell_ij(lb, tx, ti, tj);
  return {L.nx, L.ny, ti * kTW - kHalo, tj * kTH - kHalo};
}

// A thread's cells of a region W x H (with its ring) around a tile: region
// cell threadIdx.x + k kRedBlock, its place on the grid and its operator row,
// loaded at a clamped, valid index: every load of a kernel is issued before
// any is waited for, so the region costs one memory round trip.
template <int W, int H>
struct Region {
  static constexpr int N = W * H, P = (N + kRedBlock - 1) / kRedBlock;
  int g[P], gi[P], gj[P];      // cell index (0 outside the grid), place
  bool in[P], red[P];
  double d[P], ax[P], ay[P];
  __device__ __forceinline__ void load(const LevelDev &L, int i0, int j0) {
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const unsigned r = threadIdx.x + k * kRedBlock;
      const int rj = r / W, ri = r - rj * W;
      gi[k] = i0 + ri;
      gj[k] = j0 + rj;
      in[k] = (int)r < N && gi[k] >= 0 && gi[k] < L.nx && gj[k] >= 0 && gj[k] < L.ny;
      red[k] = ((gi[k] + gj[k]) & 1) == 0;
      g[k] = in[k] ? gj[k] * L.nx + gi[k] : 0;
      d[k] = L.dg[g[k]]; ax[k] = L.ax[g[k]]; ay[k] = L.ay[g[k]];
    }
  }
  // the k-th cell lies at least m cells inside the region
  __device__ __forceinline__ bool inner(int k, int m) const {
    const unsigned r = threadIdx.x + k * kRedBlock;
    const int rj = r / W, ri = r - rj * W;
    return ri >= m && ri < W - m && rj >= m && rj < H - m;
  }
  // couplings to the east and north (0 outside the grid and across its edge:
  // they are stored so) into LDS
  __device__ __forceinline__ void couplings(double *sax, double *say) const {
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const int r = threadIdx.x + k * kRedBlock;
      if (r < N) {
        sax[r] = in[k] ? ax[k] : 0.0;
        say[r] = in[k] ? ay[k] : 0.0;
      }
    }
  }
  // v + the sum of region cell r's couplings times x of its neighbours
  static __device__ __forceinline__ double add_nb(int r, const double *sax, const double *say,
                                                  const double *x, double v) {
    v = fma(sax[r], x[r + 1], v);
    v = fma(sax[r - 1], x[r - 1], v);
    v = fma(say[r], x[r + W], v);
    return fma(say[r - W], x[r - W], v);
  }
  // d x - the sum of region cell r's couplings times x of its neighbours
  static __device__ __forceinline__ double apply(int r, double d, const double *sax,
                                                 const double *say, const double *x) {
    double y = fma(d, x[r], -(sax[r] * x[r + 1]));
    y = fma(-sax[r - 1], x[r - 1], y);
    y = fma(-say[r], x[r + W], y);
    return fma(-say[r - W], x[r - W], y);
  }
};

// Bound by latency: at 256 x 256 (256 tiles) and below a launch is one round
// of short phases: one round trip to memory, then 3 half sweeps on the LDS. A
// thread keeps its region cells' places and operator in registers from the
// loads to the last half sweep (the CG update of level 0 as well) and forms
// the reciprocals of its divisions once (div64: the quotients are a division's
// bits; every operation and its order is that of the plain form, see
// launch_synth_solve on FP32-mixed plans). 128 x 128: 6.2 to 4.8 us a launch
// (k_mg_up0 4.6 to 4.0); 512 x 512: 7.7 to 6.6 (8.3 to 6.8); 1024 x 1024: 11.4
// to 10.3 (20.8 to 16.8).
__global__ void __launch_bounds__(kRedBlock) k_mg_down(const SynthDesc *ds, const int2 *bt, int l,
                                                       int v, int rr_ext) {
  __shared__ double sb[kRN], sd[kRN], sax[kRN], say[kRN], sx[kRN], sr[kTW * kTH], sh[kRedBlock];
  typedef Region<kRW, kRH> Reg;
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1], f3 = D.state[3];   // tested after the region loads
  const LevelDev L = level(D, l), CL = level(D, l + 1);
  const bool upd = l == 0 && v > 0;
  const int it = v - 1;
  double *xs = L.xs;
  const Tile T = tile_of(L, B.lb);
  // the thread's tile cell
  const int ti = threadIdx.x % kTW, tj = threadIdx.x / kTW;
  const int gi = T.i0 + kHalo + ti, gj = T.j0 + kHalo + tj;
  const bool in = gi < T.nx && gj < T.ny;
  const int g = gj * T.nx + gi;
  Reg R;
  R.load(L, T.i0, T.j0);
  double vb[Reg::P], vw[Reg::P], vs[Reg::P];
  const double *b = upd ? cg_rv(D, it) : lev_b(D, l, v);
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) vb[k] = b[R.g[k]];
  double zc = 0.0, pc0 = 0.0, xc = 0.0;
  UpdPre q = {0.0, 0.0, 1.0, 1.0};
  if (upd) {
    // r_{v-1} (in vb), w and s_old of the region, z, p and x of the tile
    // cell; p and s of iteration 0 are not there yet
    q = upd_prefetch(D, it);
    const double *w = D.cg_w, *so = it > 0 ? cg_s(D, it - 1) : w;
#pragma unroll
    for (int k = 0; k < Reg::P; ++k) { vw[k] = w[R.g[k]]; vs[k] = so[R.g[k]]; }
    const int gc = in ? g : 0;
    zc = D.cg_z[gc];
    pc0 = it > 0 ? D.cg_p[gc] : 0.0;
    xc = D.lev[0].x[gc];
  }
  // the r.r test of the CG step before this V-cycle is made by the next
  // kernel of the cycle (level 1 here, block 0; the other blocks go on: if
  // it converged, their results are not used)
  const bool fin = l == 1 && B.lb == 0 && !rr_ext;   // rr_ext: k_rr_test made it
  RRPre qr = {0.0, 0.0, 0.0};
  if (fin) qr = rr_prefetch(D, v == 0, v > 0);
  if (f1 != 0 || f3 != 0) return;
  if (fin) (void)finish_rr(D, v == 0, v > 0, sh, qr);
  double rr = 0.0;
  if (upd) {
    // the CG update: beta and alpha from the r.z and z.w partials (every
    // block sums them in the same order); s = w + beta s_old, r_v = r_{v-1} -
    // alpha s on the region; s, r_v, p = z + beta p and x += alpha p of the
    // tile to global
    const CGCoef c = upd_coef(D, B, it, q, sh);
    double *s = cg_s(D, it), *rv = cg_rv(D, v);
#pragma unroll
    for (int k = 0; k < Reg::P; ++k) {
      const double sv = it > 0 ? fma(c.be, vs[k], vw[k]) : vw[k];
      vb[k] = fma(-c.al, sv, vb[k]);
      if (R.in[k] && R.inner(k, kHalo)) {
        s[R.g[k]] = sv;
        rv[R.g[k]] = vb[k];
        rr = fma(vb[k], vb[k], rr);
      }
    }
    if (in) {
      const double pc = it > 0 ? fma(c.be, pc0, zc) : zc;
      D.cg_p[g] = pc;
      D.lev[0].x[g] = fma(c.al, pc, xc);
    }
  }
  // red half sweep from zero on the whole region
  R.couplings(sax, say);
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (r < kRN) {
      vb[k] = R.in[k] ? vb[k] : 0.0;
      R.d[k] = R.in[k] ? R.d[k] : 1.0;
      vw[k] = rcp64(R.d[k]);
      sb[r] = vb[k];
      sd[r] = R.d[k];
      sx[r] = R.red[k] ? div64(vb[k], R.d[k], vw[k]) : 0.0;
    }
  }
  __syncthreads();
  // black half sweep on the tile and a ring of one
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (!R.red[k] && R.inner(k, 1))
      sx[r] = div64(Reg::add_nb(r, sax, say, sx, vb[k]), R.d[k], vw[k]);
  }
  __syncthreads();
  // residuals; x of the tile to global
  {
    const int r = (tj + kHalo) * kRW + ti + kHalo;
    sr[threadIdx.x] = in ? sb[r] - Reg::apply(r, sd[r], sax, say, sx) : 0.0;
    if (in) xs[g] = sx[r];
  }
  if (upd) {
    const double t = block_sum(rr, sh);   // (its barriers are the restriction's)
    if (threadIdx.x == 0) red_rrt(D)[B.lb] = t;
  } else {
    __syncthreads();
  }
  // restriction: coarse cells whose children lie in this tile
  const int sx_ = L.fx >> 1, sy_ = L.fy >> 1;
  const int cw = kTW >> sx_, ch = kTH >> sy_;
  if ((int)threadIdx.x < cw * ch) {
    const int ci = threadIdx.x & (cw - 1), cj = threadIdx.x >> (5 - sx_);
    const int CI = ((T.i0 + kHalo) >> sx_) + ci, CJ = ((T.j0 + kHalo) >> sy_) + cj;
    if (CI < CL.nx && CJ < CL.ny) {
      const double *p = sr + (cj << sy_) * kTW + (ci << sx_);
      double acc = p[0];
      if (sx_) acc += p[1];
      if (sy_) acc += p[kTW];
      if (sx_ && sy_) acc += p[kTW + 1];
      CL.b[CJ * CL.nx + CI] = acc;
    }
  }
}
static_assert(kTW == 32, "the restriction's shift");

__global__ void __launch_bounds__(kRedBlock) k_mg_up(const SynthDesc *ds, const int2 *bt, int l,
                                                     int vc, double omega) {
  __shared__ double sax[kRN], say[kRN], sx[kRN], sxc[kRN];
  typedef Region<kRW, kRH> Reg;
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1], f3 = D.state[3];   // tested after the region loads
  const LevelDev L = level(D, l), CL = level(D, l + 1);
  const double *b = lev_b(D, l, vc), *xs = L.xs, *e = CL.x;
  double *x = lev_x(D, l);
  const Tile T = tile_of(L, B.lb);
  const int sx_ = L.fx >> 1, sy_ = L.fy >> 1;
  const int ti = threadIdx.x % kTW, tj = threadIdx.x / kTW;
  const int gi = T.i0 + kHalo + ti, gj = T.j0 + kHalo + tj;
  const bool in = gi < T.nx && gj < T.ny;
  const int g = in ? gj * T.nx + gi : 0;
  Reg R;
  R.load(L, T.i0, T.j0);
  double vb[Reg::P], vs[Reg::P], ve[Reg::P];
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    vb[k] = b[R.g[k]];
    vs[k] = xs[R.g[k]];
    ve[k] = e[R.in[k] ? (R.gj[k] >> sy_) * CL.nx + (R.gi[k] >> sx_) : 0];
  }
  const double bc = b[g], dc = L.dg[g];
  if (f1 != 0 || f3 != 0) return;
  // the pre-smoothed x plus the scaled coarse correction: the black half
  // sweep sees corrected red neighbours
  R.couplings(sax, say);
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (r < kRN) sxc[r] = R.in[k] ? fma(omega, ve[k], vs[k]) : 0.0;
    vb[k] = R.in[k] ? vb[k] : 0.0;
    R.d[k] = R.in[k] ? R.d[k] : 1.0;
    vs[k] = rcp64(R.d[k]);
  }
  const double ic = rcp64(dc);
  __syncthreads();
  // black half sweep on the tile and a ring of one, into sx
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (!R.red[k] && R.inner(k, 1))
      sx[r] = div64(Reg::add_nb(r, sax, say, sxc, vb[k]), R.d[k], vs[k]);
  }
  __syncthreads();
  // red half sweep on the tile with the new black neighbours
  if (in) {
    const int r = (tj + kHalo) * kRW + ti + kHalo;
    x[g] = ((gi + gj) & 1) == 0 ? div64(Reg::add_nb(r, sax, say, sx, bc), dc, ic) : sx[r];
  }
}

// Level 0 going up: as k_mg_up, over a ring of three, so that z is final on
// the tile and a ring of one (black on the tile and a ring of two, red on
// the tile and a ring of one); then w = A z on the tile, z and w to global,
// and partials of r.z and z.w for the CG (b = r).
constexpr int kU0Halo = 3, kU0W = kTW + 2 * kU0Halo, kU0H = kTH + 2 * kU0Halo;
__global__ void __launch_bounds__(kRedBlock) k_mg_up0(const SynthDesc *ds, const int2 *bt, int vc,
                                                      double omega) {
  typedef Region<kU0W, kU0H> Reg;
  __shared__ double sax[Reg::N], say[Reg::N], sxc[Reg::N], sx[Reg::N];
  __shared__ double sh[kRedBlock];
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1], f3 = D.state[3];   // tested after the region loads
  const LevelDev L = level(D, 0), CL = level(D, 1);
  const double *b = cg_rv(D, vc);
  const int nx = L.nx, ny = L.ny, sx_ = L.fx >> 1, sy_ = L.fy >> 1;
  int ti, tj;
  cell_ij(B.lb, (nx + kTW - 1) / kTW, ti, tj);
  const int i0 = ti * kTW - kU0Halo, j0 = tj * kTH - kU0Halo;
  // the thread's tile cell
  const int ci = threadIdx.x % kTW, cj = threadIdx.x / kTW;
  const int gi = i0 + kU0Halo + ci, gj = j0 + kU0Halo + cj;
  const bool in = gi < nx && gj < ny;
  const int g = in ? gj * nx + gi : 0;
  Reg R;
  R.load(L, i0, j0);
  double vb[Reg::P], vs[Reg::P], ve[Reg::P];
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    vb[k] = b[R.g[k]];
    vs[k] = L.xs[R.g[k]];
    ve[k] = CL.x[R.in[k] ? (R.gj[k] >> sy_) * CL.nx + (R.gi[k] >> sx_) : 0];
  }
  const double bc = b[g], dc = L.dg[g];
  if (f1 != 0 || f3 != 0) return;
  R.couplings(sax, say);
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (r < Reg::N) sxc[r] = R.in[k] ? fma(omega, ve[k], vs[k]) : 0.0;
    vb[k] = R.in[k] ? vb[k] : 0.0;
    R.d[k] = R.in[k] ? R.d[k] : 1.0;
    vs[k] = rcp64(R.d[k]);
  }
  __syncthreads();
  // black on the region less a ring of one, into sx
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (!R.red[k] && R.inner(k, 1))
      sx[r] = div64(Reg::add_nb(r, sax, say, sxc, vb[k]), R.d[k], vs[k]);
  }
  __syncthreads();
  // red on the region less a ring of two (reads black cells only)
#pragma unroll
  for (int k = 0; k < Reg::P; ++k) {
    const int r = threadIdx.x + k * kRedBlock;
    if (R.red[k] && R.inner(k, 2))
      sx[r] = div64(Reg::add_nb(r, sax, say, sx, vb[k]), R.d[k], vs[k]);
  }
  __syncthreads();
  // the tile cell of this thread: z, w = A z, partials of r.z and z.w
  const int r = (cj + kU0Halo) * kU0W + ci + kU0Halo;
  const double zv = in ? sx[r] : 0.0;
  const double wv = in ? Reg::apply(r, dc, sax, say, sx) : 0.0;
  if (in) {
    D.cg_z[g] = zv;
    D.cg_w[g] = wv;
  }
  // (selected, so that no product is fused into the first add of the sums)
  double trz = in ? bc * zv : 0.0, tzw = in ? zv * wv : 0.0;
  block_sum2(trz, tzw, sh);
  if (threadIdx.x == 0) {
    red_rz(D)[B.lb] = trz;
    red_zw(D)[B.lb] = tzw;
  }
}

// The coarse end of the V-cycle (every level from the first with at most
// kCoarseCells cells down to the dense solve) in one workgroup per problem,
// so the half sweeps are separated by workgroup barriers instead of kernel
// launches. Bound by latency: loads and index arithmetic until the first half
// sweep (12,000 of 25,000 cycles), then some twenty phases of 400 to 1100.
// 64 x 64 below 128 x 128: 16.7 us before, 10.7 us; 50 x 50: 16.5 to 10.1 us.
// On the way there: 13.1 us with 512 threads and pairs alone, 12.0 with the
// planes, 10.7 with the shared offsets; with 1024 threads and as much owned the
// registers spill (20 us).
//  * 512 threads with 256 registers each rather than 1024 with 128: half the
//    waves meet at a barrier, and what a thread holds once (places, the
//    dense inverse's part, the owned lower levels) it holds for twice the
//    cells.
//  * Thread t owns the top level's pairs of cells (2 p, 2 p + 1), p = t + 512
//    m: one of each colour, so no lane idles in a half sweep, and two
//    neighbouring values per load. It owns pair t of the next two levels
//    (those of at most 512 pairs). Owned operators and right-hand sides stay
//    in registers and a phase is the reads of four neighbours from LDS.
//    Levels below keep theirs in LDS. Vectors live in LDS.
//  * The top level's x lies in two planes, one per colour, cell c at c / 2.
//    The neighbours of a cell are in the other plane, at the same place, one
//    to the side and half a row up and down: neighbouring lanes read
//    neighbouring words, and with zeros around the planes no edge is a case
//    of its own.
//  * After the second (black) half sweep from zero the black residuals
//    vanish, so only red cells form one. The black cells start at 0: a
//    missing neighbour reads the cell itself, times a zero coupling, which
//    must not find what the LDS held before.
//  * Going up, the black half sweep reads its red neighbours with the
//    scaled coarse correction added (x + omega e, formed where it is read:
//    the corrected values of black cells are never read), then the red half
//    sweep recomputes the red cells, as in the tile kernels.
//  * The restriction of a level's residuals also makes the next level's
//    first (red, from zero) half sweep.
//  * Two waves share a SIMD, so 500 instructions of index arithmetic are 4000
//    cycles: addresses are 32-bit offsets shared by the arrays of a level.
constexpr int kCoarseThreads = 512;
constexpr int kCoarseCells = 8 * kCoarseThreads;

// Cell number e of colour k ((i + j) & 1 == k) of an nx x ny grid, cells of
// a colour numbered row by row. Rows come in pairs holding nx cells of each
// colour. False past the last cell of the colour.
__device__ inline bool colour_cell(int e, int k, int nx, int ny, int &i, int &j) {
  int r, p;
  cell_ij(e, nx, r, p);                     // e = p nx + r
  const int c0 = (nx + 1 - k) >> 1;         // colour-k cells of the even row
  if (r < c0) { j = 2 * p; i = k + 2 * r; }
  else { j = 2 * p + 1; i = (1 - k) + 2 * (r - c0); }
  return j < ny;
}

// Two consecutive cells of a level below the top that a thread owns, by
// colour (0 red, 1 black; in this order of cells colours alternate, also from
// one row to the next when nx is odd), and the LDS places of them and of their
// neighbours. A neighbour that does not exist is given the cell's own place,
// with a zero coupling; so has a last cell without its other one
// (right-hand side 0).
struct Pair {
  int c[2], e[2], w[2], n[2], s[2];
  int pc;                      // parent of the black cell on the next level
  int f;                       // flags below
  double d[2], id[2], aE[2], aW[2], aN[2], aS[2];
};
// kOk: the pair exists; kLB: its first (left) cell is black; kTwo: the right
// cell exists. Parents of the black cell's neighbours that differ from its
// own: kPE, kPW, kPN, kPS. kWrap: the pair across the first row's end
enum { kOk = 1, kLB = 2, kTwo = 4, kPE = 8, kPW = 16, kPN = 32, kPS = 64, kWrap = 128 };
typedef double dbl2 __attribute__((ext_vector_type(2), aligned(8)));

// The problem's record for these kernels (CoarseRec in lane k's word k): read
// by one vector load instead of a chain of scalar ones.
typedef const __attribute__((address_space(1))) double *gdbl;
typedef const __attribute__((address_space(1))) dbl2 *gdbl2;
typedef const __attribute__((address_space(1))) char *gchr;
// one or two values at a byte offset (an address register pair for the base,
// one 32-bit register for the offset)
__device__ __forceinline__ double ld1(gdbl b, unsigned o) { return *(gdbl)((gchr)b + o); }
__device__ __forceinline__ dbl2 ld2(gdbl b, unsigned o) { return *(gdbl2)((gchr)b + o); }
__device__ __forceinline__ int coarse_words(const SynthDesc *ds) {
  const int *w = (const int *)&ds[blockIdx.x].cl;
  return w[threadIdx.x & 63];
}
// margin around the top level's planes: half a row, and one
__host__ __device__ inline int coarse_margin(int nx, int ny) {
  return 1 + (ny > 1 ? (nx + 1) / 2 : 0);
}
// LDS of the top level: three margins, the planes, r
inline int coarse_top_words(int nx, int ny, bool only) {
  const int n = nx * ny, h = (n + 1) / 2;
  return 3 * coarse_margin(nx, ny) + 2 * h + (only ? n : h);
}
// A level: sizes, log2 of the aggregates, LDS offsets (doubles) of x, b, r
// and the operator (1/diag, ax, ay, diag). The top level has x, r and, between
// three margins of zeros, planes of h places, s apart,
// black after red; its r is the red plane's (in order and of both colours when
// there is no other level).
struct Lev {
  int nx, ny, n, sx, sy, x, b, r, a, h, pad, s;
};

// M: top pairs per thread; OM: owned levels below the top at most
template <int M, int OM>
struct CoarseWG {
  double *sm;
  const int hdr, tid;          // word tid & 63 of the record; thread
  const int last;              // the coarsest level
  int ol;                      // levels 1 .. ol are owned by threads
  const double omega;
  // the top level's pairs, by colour; places of the neighbours in the other
  // plane, relative to the pair's: east at te (red), 1 - te (black), west one
  // before it, north at tg (red), th (black), south at -th (red), -tg (black)
  double ti[2][M], tE[2][M], tW[2][M], tN[2][M], tS[2][M];   // 1 / diagonal, couplings
  double tb[2][M];             // right-hand side
  double td[2][M];             // diagonal
  int te[M], tg[M], th[M];
  int tij[M];                  // the left cell's i | j << 16
  Pair lo[OM];
  double lb[2][OM];
  int lch[2][OM];              // red children (two 16-bit indices, kNone)
  int dch;                     // of cell tid of level ol + 1
  double ainv[8];
  double ay0[OM + 1];          // the owned levels' first ay
  int nd;
  int lw[OM + 2][2];           // records of the top, the owned levels and the next
  gdbl ldg[OM + 1];
  Lev low, end;                // the first level not owned, the coarsest
  static constexpr int kNone = 0xffff;

  __device__ __forceinline__ CoarseWG(int h, double *s, double om)
      : sm(s), hdr(h), tid(threadIdx.x), last(word(kCwLast)), omega(om) {
#pragma unroll
    for (int t = 0; t < OM + 2; ++t) {
      lw[t][0] = word(kCwLev + 4 * t);
      lw[t][1] = word(kCwLev + 4 * t + 1);
      if (t <= OM) ldg[t] = (gdbl)ptr(kCwLev + 4 * t + 2);
    }
    const int n1 = lev(1).n, n2 = lev(2).n;
    ol = 0;
    if (OM >= 1 && last > 1 && n1 <= 2 * kCoarseThreads) ol = 1;
    if (OM >= 2 && ol == 1 && last > 2 && n2 <= 2 * kCoarseThreads) ol = 2;
    low = lev_at(ol + 1);
    end = lev_at(last);
    nd = end.n;
  }
  // The record's words come from one lane each, not from memory: read where
  // all lanes are active.
  __device__ __forceinline__ int word(int k) const { return __builtin_amdgcn_readlane(hdr, k); }
  __device__ __forceinline__ unsigned long long ptr(int k) const {
    return (unsigned long long)(unsigned)word(k) | (unsigned long long)(unsigned)word(k + 1) << 32;
  }
  static __device__ __forceinline__ Lev decode(int w0, int w1, bool first) {
    Lev l;
    l.nx = w0 & 0xffff;
    l.ny = (unsigned)w0 >> 16;
    l.n = l.nx * l.ny;
    l.sx = (w1 >> 20) & 1;
    l.sy = (w1 >> 21) & 1;
    l.x = w1 & 0xfffff;
    l.b = l.x + l.n;
    l.r = l.b + l.n;
    l.a = l.r + l.n;
    l.h = l.pad = l.s = 0;
    if (first) {
      l.h = (l.n + 1) >> 1;
      l.pad = coarse_margin(l.nx, l.ny);
      l.s = l.h + l.pad;
      l.r = l.x + 2 * l.s + l.pad;
      l.x += l.pad;
    }
    return l;
  }
  __device__ __forceinline__ Lev lev(int t) const {   // t known at compile time, <= OM + 1
    if (t > OM + 1) return lev_at(t);
    return decode(lw[t][0], lw[t][1], t == 0);
  }
  __device__ __forceinline__ Lev lev_at(int t) const {
    return decode(word(kCwLev + 4 * t), word(kCwLev + 4 * t + 1), t == 0);
  }

  __device__ __forceinline__ RRTest rr_test(bool first, bool tiles, int32_t *state) const {
    const int nb = word(kCwNb);
    const double *red = (const double *)(gdbl)ptr(kCwRed);
    RRTest T;
    T.rr = tiles ? red + word(kCwRrt) : red;
    T.nrr = tiles ? word(kCwTile) : nb;
    T.bb = red + nb;
    T.nb = nb;
    T.first = first;
    T.scal = (double *)(__attribute__((address_space(1))) double *)ptr(kCwScal);
    T.state = state;
    T.rtol = __longlong_as_double((long long)ptr(kCwRtol));
    return T;
  }

  // Pair p of level t > 0, its left cell at (i, j): loads of the operator, by
  // place (left 0, right 1) until sort() orders them by colour, and the places
  // meanwhile. Couplings across a grid's edge are stored as zeros (ax at the
  // end of each row, ay on the last row): those of the west and south edges
  // are read there (coarse_places.h: also what loads one value past an array).
  __device__ __forceinline__ void own(Pair &q, int t, int p, int i, int j) {
    const Lev v = lev(t);
    const int nx = v.nx, ny = v.ny, n = v.n, l = 2 * p;
    const gdbl dg = ldg[t], ax = dg + op_ax(n), ay = dg + op_ay(n);
    const bool W = i > 0, SL = j > 0;
    const unsigned o = 8u * l;
    const dbl2 d = ld2(dg, o), x = ld2(ax, o), y = ld2(ay, o);
    const dbl2 u = ld2(ay, o + 8u * south_step(j, nx, n));
    q.aW[0] = ld1(ax, o + 8u * west_step(i, nx));
    q.d[0] = d.x; q.d[1] = d.y;
    q.aE[0] = q.aW[1] = x.x; q.aE[1] = x.y;
    q.aN[0] = y.x; q.aN[1] = y.y;
    q.aS[0] = u.x; q.aS[1] = u.y;
    const bool in = i + 1 < nx, two = l + 1 < n;   // in: both in one row
    const int ir = in ? i + 1 : 0, jr = in ? j : j + 1;
    const bool ER = two && ir + 1 < nx, EL = two && in, SR = two && jr > 0;
    const bool NL = j + 1 < ny, NR = two && jr + 1 < ny, lbk = (i + j) & 1;
    const int r = two ? l + 1 : l;
    const int eL = EL ? 1 : 0, eR = ER ? 1 : 0, wL = W ? 1 : 0;
    const int nL = NL ? nx : 0, nR = NR ? nx : 0, sL = SL ? nx : 0, sR = SR ? nx : 0;
    q.c[0] = lbk ? r : l; q.c[1] = lbk ? l : r;
    q.e[0] = q.c[0] + (lbk ? eR : eL); q.e[1] = q.c[1] + (lbk ? eL : eR);
    q.w[0] = q.c[0] - (lbk ? eL : wL); q.w[1] = q.c[1] - (lbk ? wL : eL);
    q.n[0] = q.c[0] + (lbk ? nR : nL); q.n[1] = q.c[1] + (lbk ? nL : nR);
    q.s[0] = q.c[0] - (lbk ? sR : sL); q.s[1] = q.c[1] - (lbk ? sL : sR);
    q.f = kOk | (lbk ? kLB : 0) | (two ? kTwo : 0) | (!in && !SL ? kWrap : 0);
    // with aggregates of two, the odd cell's next and the even cell's
    // previous neighbour have another parent; of one, every neighbour
    const int sx = v.sx, sy = v.sy, cnx = lev(t + 1).nx;
    const int ib = lbk ? i : ir, jb = lbk ? j : jr;
    const bool N = lbk ? NL : NR, S = lbk ? SL : SR, E = lbk ? EL : ER, Wb = lbk ? W : EL;
    q.pc = lbk || two ? (jb >> sy) * cnx + (ib >> sx) : 0;
    const bool xo = !sx || (ib & 1), xe = !sx || !(ib & 1);
    const bool yo = !sy || (jb & 1), ye = !sy || !(jb & 1);
    q.f |= (E && xo ? kPE : 0) | (Wb && xe ? kPW : 0) | (N && yo ? kPN : 0) | (S && ye ? kPS : 0);
  }
  // the loaded operator by colour (a missing cell has none), the diagonal
  // inverted
  __device__ __forceinline__ void sort(Pair &q, int t) {
    const bool lbk = q.f & kLB, two = q.f & kTwo;
    const double el = q.aE[0], er = two ? q.aE[1] : 0.0, wl = q.aW[0], wr = two ? q.aW[1] : 0.0;
    const double nl = q.aN[0], nr = two ? q.aN[1] : 0.0, sl = q.aS[0];
    const double sr = !two ? 0.0 : q.f & kWrap ? ay0[t] : q.aS[1];
    const double dl = q.d[0], dr = two ? q.d[1] : 1.0;
    q.aE[0] = lbk ? er : el; q.aE[1] = lbk ? el : er;
    q.aW[0] = lbk ? wr : wl; q.aW[1] = lbk ? wl : wr;
    q.aN[0] = lbk ? nr : nl; q.aN[1] = lbk ? nl : nr;
    q.aS[0] = lbk ? sr : sl; q.aS[1] = lbk ? sl : sr;
    q.d[0] = lbk ? dr : dl;
    q.d[1] = lbk ? dl : dr;
    q.id[0] = div64(1.0, q.d[0], rcp64(q.d[0]));
    q.id[1] = div64(1.0, q.d[1], rcp64(q.d[1]));
  }
  // The top level's pairs: loads as for own() and, where b is not NULL, of
  // the right-hand side (a thread without an m-th pair loads pair 0).
  __device__ __forceinline__ void own_top(gdbl b) {
    const Lev v = lev(0);
    const int nx = v.nx, n = v.n;
    const gdbl dg = ldg[0], ax = dg + op_ax(n), ay = dg + op_ay(n);
    // the left cell of pair tid, and the step to that of pair tid + 512: in
    // pairs of an even row, in cells of an odd one
    const int odd = nx & 1, u = odd ? nx : nx >> 1, ha = v.ny > 1 ? nx >> 1 : 0;
    const int hb = v.ny > 1 ? nx - ha : 0;
    int r, j, dr, dj;
    cell_ij(tid << odd, u, r, j);
    cell_ij(kCoarseThreads << odd, u, dr, dj);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int p = tid + m * kCoarseThreads;
      const int i = odd ? r : 2 * r;
      const unsigned o = p < v.h ? 16u * p : 0u;
      const int ii = p < v.h ? i : 0, jj = p < v.h ? j : 0;
      const dbl2 d = ld2(dg, o), x = ld2(ax, o), y = ld2(ay, o);
      const dbl2 w = ld2(ay, o + 8u * south_step(jj, nx, n));
      tW[0][m] = ld1(ax, o + 8u * west_step(ii, nx));
      dbl2 bb = {0.0, 0.0};
      if (b) bb = ld2(b, o);
      ti[0][m] = d.x; ti[1][m] = d.y;
      tE[0][m] = tW[1][m] = x.x; tE[1][m] = x.y;
      tN[0][m] = y.x; tN[1][m] = y.y;
      tS[0][m] = w.x; tS[1][m] = w.y;
      tb[0][m] = bb.x; tb[1][m] = bb.y;
      const bool lbk = (i + j) & 1;
      tij[m] = i | j << 16;
      te[m] = lbk ? 1 : 0;
      tg[m] = lbk ? hb : ha;
      th[m] = lbk ? ha : hb;
      r += dr;
      j += dj;
      if (r >= u) { r -= u; ++j; }
    }
    ay0[0] = ld1(ay, 0);
  }
  __device__ __forceinline__ void sort_top() {
    const Lev v = lev(0);
    if (v.nx & 1) {
      // a last cell without its other one; the pair across the first row's
      // end, whose right cell's south coupling is the first of ay
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int p = tid + m * kCoarseThreads;
        if (2 * p == v.nx - 1) tS[1][m] = ay0[0];
        if (2 * p + 1 >= v.n) {
          tE[1][m] = tN[1][m] = tS[1][m] = tb[1][m] = 0.0;
          ti[1][m] = 1.0;
        }
      }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const bool lbk = te[m];
      auto by_colour = [&](double (&a)[2][M]) {
        const double l = a[0][m], r = a[1][m];
        a[0][m] = lbk ? r : l;
        a[1][m] = lbk ? l : r;
      };
      by_colour(tE);
      by_colour(tW);
      by_colour(tN);
      by_colour(tS);
      by_colour(tb);
      by_colour(ti);
      td[0][m] = ti[0][m];
      td[1][m] = ti[1][m];
      ti[0][m] = div64(1.0, td[0][m], rcp64(td[0][m]));
      ti[1][m] = div64(1.0, td[1][m], rcp64(td[1][m]));
    }
  }
  __device__ __forceinline__ bool has(int m) const {
    return tid + m * kCoarseThreads < lev(0).h;
  }
  // the place of the pair's cell of colour k
  __device__ __forceinline__ double *at(int k, int m) const {
    const Lev v = lev(0);
    return sm + v.x + (k ? v.s : 0) + tid + m * kCoarseThreads;
  }
  // the pair's cell of colour k, and whether it exists
  __device__ __forceinline__ int cell(int k, int m) const {
    return 2 * (tid + m * kCoarseThreads) + (te[m] ? 1 - k : k);
  }
  __device__ __forceinline__ bool ok(int k, int m) const { return cell(k, m) < lev(0).n; }
  // A x of an owned cell, x of the grid in LDS
  __device__ __forceinline__ double apply(int k, int m) const {
    return -add_top(k, m, -td[k][m] * *at(k, m));
  }
  // s + sum of the couplings of the top pair's cell of colour k times x
  __device__ __forceinline__ double add_top(int k, int m, double s) const {
    const double *x = at(1 - k, m), *xe = x + (k ? 1 - te[m] : te[m]);
    const double a = xe[0], b = xe[-1];
    const double n = x[k ? th[m] : tg[m]], u = x[-(k ? tg[m] : th[m])];
    s = fma(tE[k][m], a, s);
    s = fma(tW[k][m], b, s);
    s = fma(tN[k][m], n, s);
    return fma(tS[k][m], u, s);
  }
  // the same for the black cell with the scaled correction of the parents
  // (e, on the next level) added to x
  __device__ __forceinline__ double add_top_corr(int m, const double *e, double s) const {
    const Lev v = lev(0), w = lev(1);
    const double *x = at(0, m), *xp = x + 1 - te[m];
    const double xe = xp[0], xw = xp[-1], xn = x[th[m]], xs = x[-tg[m]];
    int i = tij[m] & 0xffff, j = tij[m] >> 16;
    if (!te[m]) ++i;
    if (i >= v.nx) { i = 0; j = min(j + 1, v.ny - 1); }
    // parents of the neighbours (of one within the grid where there is none)
    const int I = i >> v.sx, row = (j >> v.sy) * w.nx;
    const int ie = min((i + 1) >> v.sx, w.nx - 1), iw = max(i - 1, 0) >> v.sx;
    const int jn = min((j + 1) >> v.sy, w.ny - 1), js = max(j - 1, 0) >> v.sy;
    const double ee = e[row + ie], ew = e[row + iw], en = e[jn * w.nx + I], es = e[js * w.nx + I];
    s = fma(tE[1][m], fma(omega, ee, xe), s);
    s = fma(tW[1][m], fma(omega, ew, xw), s);
    s = fma(tN[1][m], fma(omega, en, xn), s);
    return fma(tS[1][m], fma(omega, es, xs), s);
  }
  // x of the pair's cell k on an owned level below the top (not of a missing
  // cell: it has the other one's place)
  __device__ __forceinline__ void put(double *x, const Pair &q, int k, double v) {
    if ((q.f & kTwo) || k == (q.f & kLB ? 1 : 0)) x[q.c[k]] = v;
  }
  // s + sum of the couplings of the pair's cell k times x of its neighbours
  __device__ __forceinline__ double add_nb(const Pair &q, int k, const double *x, double s) {
    const double a = x[q.e[k]], b = x[q.w[k]], n = x[q.n[k]], u = x[q.s[k]];
    s = fma(q.aE[k], a, s);
    s = fma(q.aW[k], b, s);
    s = fma(q.aN[k], n, s);
    return fma(q.aS[k], u, s);
  }
  // the same for the black cell with the scaled correction e of the parents
  // added to x
  __device__ __forceinline__ double add_nb_corr(const Pair &q, int cnx, const double *x,
                                                const double *e, double s) {
    const double xe = x[q.e[1]], xw = x[q.w[1]], xn = x[q.n[1]], xs = x[q.s[1]];
    const double ee = e[q.pc + (q.f & kPE ? 1 : 0)], ew = e[q.pc - (q.f & kPW ? 1 : 0)];
    const double en = e[q.pc + (q.f & kPN ? cnx : 0)], es = e[q.pc - (q.f & kPS ? cnx : 0)];
    s = fma(q.aE[1], fma(omega, ee, xe), s);
    s = fma(q.aW[1], fma(omega, ew, xw), s);
    s = fma(q.aN[1], fma(omega, en, xn), s);
    return fma(q.aS[1], fma(omega, es, xs), s);
  }
  // the red children on level v (first: the top) of cell (I, J) of the next
  static __device__ __forceinline__ int red_children(const Lev &v, bool first, int I, int J) {
    const int nx = v.nx, ny = v.ny, fx = 1 + v.sx, fy = 1 + v.sy;
    const int i = fx * I, j = fy * J;
    int a = kNone, b = kNone;
    if (!((i + j) & 1)) {
      a = j * nx + i;
      if (fx > 1 && fy > 1 && i + 1 < nx && j + 1 < ny) b = a + nx + 1;
    } else {                   // fx or fy is 1: the other child is red
      if (fx > 1 && i + 1 < nx) a = j * nx + i + 1;
      if (fy > 1 && j + 1 < ny) a = (j + 1) * nx + i;
    }
    if (first) {               // the residuals of the red plane only
      if (a != kNone) a >>= 1;
      if (b != kNone) b >>= 1;
    }
    return a | b << 16;
  }
  __device__ __forceinline__ double child_sum(int ch, const double *r) {
    const unsigned a = ch & 0xffff, b = (unsigned)ch >> 16;
    const double u = r[a != kNone ? a : 0], v = r[b != kNone ? b : 0];
    const double s = a != kNone ? u : 0.0;
    return b != kNone ? s + v : s;
  }

  // Loads of the owned levels (of the top right-hand side where b is not
  // NULL) and of the dense inverse, and the places while they are under way.
  __device__ __forceinline__ void begin(gdbl b) {
    own_top(b);
#pragma unroll
    for (int t = 1; t <= OM; ++t) {
      if (t > ol) break;
      const Lev v = lev(t), u = lev(t - 1);
      Pair &q = lo[t - 1];
      q.f = 0;
      ay0[t] = ld1(ldg[t], 8u * op_ay(v.n));
      if (2 * tid < v.n) {
        int i, j;
        cell_ij(2 * tid, v.nx, i, j);
        own(q, t, tid, i, j);
        const bool in = i + 1 < v.nx, lbk = q.f & kLB;
        const int cl = red_children(u, t == 1, i, j);
        const int cr = q.f & kTwo
                           ? red_children(u, t == 1, in ? i + 1 : 0, in ? j : j + 1) : -1;
        lch[0][t - 1] = lbk ? cr : cl;
        lch[1][t - 1] = lbk ? cl : cr;
      }
    }
    // the coarsest level's dense inverse (n <= 64): 8 threads per row (terms
    // past the row's end are dropped where they are used)
    const gdbl Ainv = (gdbl)ptr(kCwInv);
    {
      const int a = (tid >> 3) * nd + (tid & 7), e = nd * nd - 1;
#pragma unroll
      for (int q = 0; q < 8; ++q) ainv[q] = ld1(Ainv, 8u * min(a + 8 * q, e));
    }
    dch = -1;
    if (last > 0) {
      const Lev u = lev_at(ol);
      const bool first = ol == 0;
      if (tid < low.n) {
        int i, j;
        cell_ij(tid, low.nx, i, j);
        dch = red_children(u, first, i, j);
      }
    }
  }
  // What was loaded put in place (a barrier before others' LDS).
  __device__ __forceinline__ void settle() {
    // deeper levels' operators into LDS (reciprocal diagonal, ax, ay, diagonal)
    for (int t = ol + 1; t < last; ++t) {
      const Lev v = lev_at(t);
      const int n = v.n;
      const gdbl dg = (gdbl)ptr(kCwLev + 4 * t + 2);
      double *a = sm + v.a;
      for (int c = tid; c < n; c += kCoarseThreads) {
        const double d = dg[c], x = dg[op_ax(n) + c], y = dg[op_ay(n) + c];
        a[c] = div64(1.0, d, rcp64(d)); a[n + c] = x; a[2 * n + c] = y; a[3 * n + c] = d;
      }
    }
    // the margins of the top level's planes
    const Lev v = lev(0);
    for (int c = tid; c < v.pad; c += kCoarseThreads) {
      double *x = sm + v.x - v.pad + c;
      x[0] = x[v.s] = x[2 * v.s] = 0.0;
    }
    sort_top();
#pragma unroll
    for (int t = 1; t <= OM; ++t) {
      if (t > ol) break;
      sort(lo[t - 1], t);
    }
  }

  // level t > ol: half sweep of colour k over the colour's cells
  __device__ __forceinline__ void low_half(int t, int k) {
    const Lev v = lev_at(t);
    const int nx = v.nx, ny = v.ny, n = v.n;
    double *x = sm + v.x;
    const double *b = sm + v.b, *id = sm + v.a, *ax = id + n, *ay = id + 2 * n;
    for (int e = tid; 2 * e < n + 1; e += kCoarseThreads) {
      int i, j;
      if (!colour_cell(e, k, nx, ny, i, j)) break;
      const int c = j * nx + i;
      double s = b[c];
      if (i + 1 < nx) s = fma(ax[c], x[c + 1], s);
      if (i > 0) s = fma(ax[c - 1], x[c - 1], s);
      if (j + 1 < ny) s = fma(ay[c], x[c + nx], s);
      if (j > 0) s = fma(ay[c - nx], x[c - nx], s);
      x[c] = s * id[c];
    }
  }
  // level t > ol: black half sweep with the correction of its red neighbours
  __device__ __forceinline__ void low_black_corr(int t) {
    const Lev v = lev_at(t), w = lev_at(t + 1);
    const int nx = v.nx, ny = v.ny, n = v.n, sx = v.sx, sy = v.sy, cnx = w.nx;
    double *x = sm + v.x;
    const double *e = sm + w.x;
    const double *b = sm + v.b, *id = sm + v.a, *ax = id + n, *ay = id + 2 * n;
    auto xc = [&](int i, int j) {
      return fma(omega, e[(j >> sy) * cnx + (i >> sx)], x[j * nx + i]);
    };
    for (int q = tid; 2 * q < n + 1; q += kCoarseThreads) {
      int i, j;
      if (!colour_cell(q, 1, nx, ny, i, j)) break;
      const int c = j * nx + i;
      double s = b[c];
      if (i + 1 < nx) s = fma(ax[c], xc(i + 1, j), s);
      if (i > 0) s = fma(ax[c - 1], xc(i - 1, j), s);
      if (j + 1 < ny) s = fma(ay[c], xc(i, j + 1), s);
      if (j > 0) s = fma(ay[c - nx], xc(i, j - 1), s);
      x[c] = s * id[c];
    }
  }
  // level v below the owned ones: residual of cell c
  __device__ __forceinline__ double low_resid(const Lev &v, int c) {
    const int nx = v.nx, ny = v.ny, n = v.n;
    const double *x = sm + v.x, *b = sm + v.b, *id = sm + v.a, *ax = id + n, *ay = id + 2 * n;
    const double *dg = id + 3 * n;
    int i, j;
    cell_ij(c, nx, i, j);
    double q = b[c];
    if (i + 1 < nx) q = fma(ax[c], x[c + 1], q);
    if (i > 0) q = fma(ax[c - 1], x[c - 1], q);
    if (j + 1 < ny) q = fma(ay[c], x[c + nx], q);
    if (j > 0) q = fma(ay[c - nx], x[c - nx], q);
    return fma(-dg[c], x[c], q);
  }
  // restriction of a level's residuals (the red ones: black residuals vanish;
  // r) to level t and, above the coarsest, its red half sweep from zero. To
  // an owned level:
  __device__ __forceinline__ void restrict_to_own(const double *r, int t, const Pair &q,
                                                  const int (&ch)[2], double &b0, double &b1) {
    double *x = sm + lev(t).x;
    if (!(q.f & kOk)) return;
    b0 = child_sum(ch[0], r);
    b1 = child_sum(ch[1], r);
    put(x, q, 0, b0 * q.id[0]);
    put(x, q, 1, 0.0);
  }
  // from the last owned level (or the top) to the next
  __device__ __forceinline__ void restrict_to_lds() {
    const Lev u = lev_at(ol);
    double *cb = sm + low.b, *cx = sm + low.x;
    const double *cid = sm + low.a, *r = sm + u.r;
    const bool sweep = ol + 1 < last, first = ol == 0;
    for (int C = tid; C < low.n; C += kCoarseThreads) {
      int I, J, ch = dch;
      cell_ij(C, low.nx, I, J);
      if (C != tid) ch = red_children(u, first, I, J);
      const double v = child_sum(ch, r);
      cb[C] = v;
      if (sweep) cx[C] = ((I + J) & 1) == 0 ? v * cid[C] : 0.0;
    }
  }
  // from level t to the next, both below them
  __device__ __forceinline__ void low_restrict(int t) {
    const Lev u = lev_at(t), w = lev_at(t + 1);
    double *cb = sm + w.b, *cx = sm + w.x;
    const double *cid = sm + w.a;
    const bool sweep = t + 1 < last;
    for (int C = tid; C < w.n; C += kCoarseThreads) {
      int I, J;
      cell_ij(C, w.nx, I, J);
      const int ch = red_children(u, false, I, J), a = ch & 0xffff, b = (unsigned)ch >> 16;
      double v = 0.0;
      if (a != kNone) v += low_resid(u, a);
      if (b != kNone) v += low_resid(u, b);
      cb[C] = v;
      if (sweep) cx[C] = ((I + J) & 1) == 0 ? v * cid[C] : 0.0;
    }
  }
  // x = M^{-1} tb on the top level: each thread's own cells (a barrier before others')
  __device__ __forceinline__ void cycle() {
    const Lev v0 = lev(0), v1 = lev(1);
    double *r0 = sm + v0.r;
    const double *x1 = sm + v1.x;
    if (last == 0) {
      // the top level is the coarsest: dense solve only (r in order)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int l = 2 * (tid + m * kCoarseThreads);
        const bool lbk = te[m];
        if (l < v0.n) r0[l] = tb[lbk ? 1 : 0][m];
        if (l + 1 < v0.n) r0[l + 1] = tb[lbk ? 0 : 1][m];
        if (has(m)) *at(0, m) = *at(1, m) = 0.0;   // also the place of a missing cell
      }
      __syncthreads();
    } else {
      // ---- down: red from zero, black, red residuals, restrict
#pragma unroll
      for (int m = 0; m < M; ++m) {
        if (!has(m)) continue;
        *at(0, m) = tb[0][m] * ti[0][m];
        *at(1, m) = 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < M; ++m)
        if (has(m)) *at(1, m) = add_top(1, m, tb[1][m]) * ti[1][m];
      __syncthreads();
#pragma unroll
      for (int m = 0; m < M; ++m)
        if (has(m))
          r0[tid + m * kCoarseThreads] = fma(-td[0][m], *at(0, m), add_top(0, m, tb[0][m]));
      __syncthreads();
#pragma unroll
      for (int t = 1; t <= OM; ++t) {
        if (t > ol) break;
        const Pair &q = lo[t - 1];
        const int ch[2] = {lch[0][t - 1], lch[1][t - 1]};
        double &b0 = lb[0][t - 1], &b1 = lb[1][t - 1];
        const Lev v = lev(t);
        double *x = sm + v.x, *r = sm + v.r;
        restrict_to_own(t == 1 ? r0 : sm + lev(t - 1).r, t, q, ch, b0, b1);
        __syncthreads();
        if (q.f & kOk) put(x, q, 1, add_nb(q, 1, x, b1) * q.id[1]);
        __syncthreads();
        if (q.f & kOk) r[q.c[0]] = fma(-q.d[0], x[q.c[0]], add_nb(q, 0, x, b0));
        __syncthreads();
      }
      restrict_to_lds();
      __syncthreads();
      for (int t = ol + 1; t < last; ++t) {
        low_half(t, 1);
        __syncthreads();
        low_restrict(t);
        __syncthreads();
      }
    }
    // ---- dense solve on the coarsest level: 8 threads per row
    {
      const double *b = last == 0 ? r0 : sm + end.b;
      double *xl = sm + end.x;
      const int row = tid >> 3, col0 = tid & 7;
      double bv[8], v = 0.0, v1 = 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) bv[q] = b[col0 + 8 * q < nd ? col0 + 8 * q : 0];
#pragma unroll
      for (int q = 0; q < 8; q += 2) {
        v = fma(ainv[q], col0 + 8 * q < nd ? bv[q] : 0.0, v);
        v1 = fma(ainv[q + 1], col0 + 8 * q + 8 < nd ? bv[q + 1] : 0.0, v1);
      }
      v += v1;
      v += __shfl_xor(v, 4, 64);
      v += dpp_d<0x4E>(v);     // lane ^ 2, lane ^ 1
      v += dpp_d<0xB1>(v);
      int at = row;
      if (last == 0) {         // the top level's place
        int i, j;
        cell_ij(row, v0.nx, i, j);
        at = ((i + j) & 1 ? v0.s : 0) + (row >> 1);
      }
      if (col0 == 0 && row < nd) xl[at] = v;
      __syncthreads();
    }
    // ---- up
    if (last == 0) return;
    for (int t = last - 1; t > ol; --t) {
      low_black_corr(t);
      __syncthreads();
      low_half(t, 0);
      __syncthreads();
    }
#pragma unroll
    for (int t = OM; t >= 1; --t) {
      if (t > ol) continue;
      const Pair &q = lo[t - 1];
      const Lev v = lev(t), w = lev(t + 1);
      double *x = sm + v.x;
      const double *e = sm + w.x;
      if (q.f & kOk) put(x, q, 1, add_nb_corr(q, w.nx, x, e, lb[1][t - 1]) * q.id[1]);
      __syncthreads();
      if (q.f & kOk) put(x, q, 0, add_nb(q, 0, x, lb[0][t - 1]) * q.id[0]);
      __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (has(m)) *at(1, m) = add_top_corr(m, x1, tb[1][m]) * ti[1][m];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (has(m)) *at(0, m) = add_top(0, m, tb[0][m]) * ti[0][m];
  }
};

// Sums of two values over the workgroup: wave sums, then in wave order (sh: two
// entries per wave; barriers before and between).
__device__ __forceinline__ void coarse_sum2(double &u, double &v, double *sh) {
  const double a = wave_sum(u), b = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    sh[2 * (threadIdx.x >> 6)] = a;
    sh[2 * (threadIdx.x >> 6) + 1] = b;
  }
  __syncthreads();
  u = v = 0.0;
  for (int k = 0; k < kCoarseThreads / 64; ++k) { u += sh[2 * k]; v += sh[2 * k + 1]; }
}
// The r.r test (finish_rr) of a problem that k_cg_small solves when it is alone,
// on the right-hand side in its owners' registers: the sums in k_cg_small's order.
template <class WG>
__device__ __forceinline__ bool coarse_rr(const WG &W, CDesc &D, const RRTest &T, double *sh) {
  constexpr int M = sizeof(W.te) / sizeof(W.te[0]);
  double rr = 0.0, bb = 0.0, stop = T.scal[S_STOP];
  const double *rhs = D.rhs;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (!W.ok(k, m)) continue;
      rr = fma(W.tb[k][m], W.tb[k][m], rr);
      const double b = T.first ? rhs[W.cell(k, m)] : 0.0;
      bb = fma(b, b, bb);
    }
  coarse_sum2(rr, bb, sh);
  if (T.first) stop = fmax(T.rtol * T.rtol * rr, 1e-28 * bb);
  const bool conv = !(rr > stop);
  if (threadIdx.x == 0) {
    double *scal = T.scal;
    scal[S_RR] = rr;
    if (T.first) {
      scal[S_BB] = bb;
      scal[S_STOP] = stop;
    }
    const double nit = T.first ? 0.0 : scal[S_NIT] + 1.0;
    scal[S_NIT] = nit;
    if (conv) T.state[3] = 1 + (int32_t)nit;
  }
  return conv;
}
// w = A z of CG iteration it (z: the cycle's result in LDS) and the iteration's
// coefficients, for k_cg_update, as k_cg_small forms them.
template <class WG>
__device__ __forceinline__ void coarse_zw(const WG &W, CDesc &D, int it, double *sh) {
  constexpr int M = sizeof(W.te) / sizeof(W.te[0]);
  double ga = 0.0, de = 0.0, *w = D.cg_w;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (!W.ok(k, m)) continue;
      const double wv = W.apply(k, m), z = *W.at(k, m);
      w[W.cell(k, m)] = wv;
      ga = fma(W.tb[k][m], z, ga);
      de = fma(z, wv, de);
    }
  coarse_sum2(ga, de, sh);
  if (threadIdx.x != 0) return;
  double *scal = D.scal;
  const CGCoef q = cg_coef(it == 0, ga, de, it > 0 ? scal[rz_slot(it - 1)] : 1.0,
                           it > 0 ? scal[alpha_slot(it - 1)] : 1.0);
  scal[rz_slot(it)] = ga;
  scal[alpha_slot(it)] = q.al;
  scal[S_BETA] = q.be;
  scal[S_ZW] = de;
}

// SUMS: some problem of the set has kCoefCoarse (batches; the code for it takes
// registers that M = 4 does not have to spare).
template <int M, bool SUMS>
__global__ void __launch_bounds__(kCoarseThreads) k_mg_coarse(const SynthDesc *ds, double omega,
                                                              int vc, int rr_ext) {
  extern __shared__ double sm[];
  __shared__ double red[2 * kCoarseThreads / 64];
  CoarseWG<M, 2> W(coarse_words(ds), sm, omega);
  // a problem whose V-cycle starts here or on level 1 makes the r.r test of
  // the CG step before it here (level 1: the level-0 tile kernel made the
  // update)
  const int lc = W.word(kCwLc);
  // (a problem that k_cg_small solves alone: below, in its order)
  const bool sums = SUMS && W.word(kCwSums) != 0;
  const bool fin = !sums && (lc == 0 || (lc == 1 && !rr_ext));   // rr_ext: k_rr_test made it
  const RRTest T = W.rr_test(vc == 0, vc > 0 && lc == 1, cdesc(ds, blockIdx.x).state);
  RRPre q = {0.0, 0.0, 0.0};
  if (fin) q = rr_prefetch(T);
  const int32_t f1 = T.state[1], f3 = T.state[3];   // tested after the loads are issued
  W.begin((gdbl)W.ptr(vc & 1 ? kCwB1 : kCwB0));
  if (f1 != 0 || f3 != 0) return;
  if (fin && finish_rr(T, red, q)) return;
  W.settle();
  if constexpr (SUMS)
    if (sums && coarse_rr(W, cdesc(ds, blockIdx.x), T, red)) return;
  W.cycle();
  if constexpr (SUMS)
    if (sums) coarse_zw(W, cdesc(ds, blockIdx.x), vc, red);
  // x of the top level (when that is level 0, k_cg_zw then forms w = A z and
  // the CG's partials)
  double *xout = (double *)(__attribute__((address_space(1))) double *)W.ptr(kCwX);
  const int n = W.lev(0).n;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int c = 2 * ((int)threadIdx.x + m * kCoarseThreads);
    if (!W.has(m)) continue;
    const bool lb = W.te[m];
    const double u = *W.at(0, m), v = *W.at(1, m), l = lb ? v : u, r = lb ? u : v;
    if (c + 1 < n) *(dbl2 *)(xout + c) = dbl2{l, r};
    else xout[c] = l;
  }
}

// For a problem whose whole V-cycle ran in the one-workgroup kernel: w = A z
// and partials of r.z and z.w per block of cells (r of V-cycle vc).
__global__ void k_cg_zw(const SynthDesc *ds, const int2 *bt, int vc) {
  __shared__ double sh[kRedBlock];
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  if (D.lc > 0 || D.coef_sep == kCoefCoarse) return;
  const int32_t f1 = D.state[1], f3 = D.state[3];
  const LevelDev L = level(D, 0);
  const int nx = L.nx, ny = L.ny;
  const int c = B.lb * kRedBlock + threadIdx.x;
  const bool in = c < D.N;
  int i = 0, j = 0;
  if (in) cell_ij(c, nx, i, j);
  const bool hE = in && i + 1 < nx, hW = in && i > 0, hN = in && j + 1 < ny, hS = in && j > 0;
  const int cc = in ? c : 0;
  const double *z = D.cg_z;
  const double zc = z[cc], ze = z[hE ? c + 1 : cc], zw = z[hW ? c - 1 : cc];
  const double zn = z[hN ? c + nx : cc], zs = z[hS ? c - nx : cc];
  const double dg = L.dg[cc], aE = L.ax[cc], aW = L.ax[hW ? c - 1 : cc];
  const double aN = L.ay[cc], aS = L.ay[hS ? c - nx : cc];
  const double rc = cg_rv(D, vc)[cc];
  if (f1 != 0 || f3 != 0) return;
  double wv = dg * zc;
  if (hE) wv -= aE * ze;
  if (hW) wv -= aW * zw;
  if (hN) wv -= aN * zn;
  if (hS) wv -= aS * zs;
  if (in) D.cg_w[c] = wv;
  const double trz = block_sum(in ? rc * zc : 0.0, sh);
  const double tzw = block_sum(in ? zc * wv : 0.0, sh);
  if (threadIdx.x == 0) {
    red_rz(D)[B.lb] = trz;
    red_zw(D)[B.lb] = tzw;
  }
}


constexpr double kOmega = 1.7;   // coarse-grid correction scaling (aggregation MG)

// The whole synthetic solve of a problem of at most kCoarseCells cells in one
// workgroup (launch_synth_solve's iteration, with the same stop test): the
// CG's vectors stay with the cells' owners in registers, the operators are
// loaded once, and neither a launch nor the host stands between two
// iterations. As separate kernels an iteration was four launches of 3 to 7 us
// and the solve a wait of the host: 32 x 32, two iterations a solve, 45 us of
// kernels, here 13.4 us. Outer iterations in all, before and here: 40 x 40 88
// to 55 us, 50 x 50 92 to 72 (80 with four pairs per thread for its three), 64 x
// 64 121 to 108 (four pairs: the CG's vectors spill).
// MODE: see k_cg_begin.
template <int M, int MODE>
__global__ void __launch_bounds__(kCoarseThreads) k_cg_small(const SynthDesc *ds, int sub,
                                                             int max_it) {
  extern __shared__ double sm[];
  __shared__ double red[2 * kCoarseThreads / 64];
  CDesc &D = cdesc(ds, blockIdx.x);
  if (D.state[1] != 0) return;
  CoarseWG<M, M >= 3 ? 1 : 2> W(coarse_words(ds), sm, kOmega);
  W.begin(nullptr);
  W.settle();
  const int nx = D.nx;
  double *xg = D.lev[0].x;
  const double *X = MODE >= 2 ? xg : D.phi;
  double x[2][M], p[2][M], s[2][M];
  double (&r)[2][M] = W.tb;        // the residual is the V-cycle's right-hand side
  auto sum2 = [&](double &u, double &v) { coarse_sum2(u, v, red); };
  auto cell = [&](int k, int m) { return W.cell(k, m); };
  auto ok = [&](int k, int m) { return cell(k, m) < D.N; };
  auto apply = [&](int k, int m) { return W.apply(k, m); };
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      x[k][m] = ok(k, m) ? X[cell(k, m)] : 0.0;
      p[k][m] = s[k][m] = 0.0;
      if (W.has(m)) *W.at(k, m) = x[k][m];
    }
  __syncthreads();
  double rr = 0.0, bb = 0.0;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      r[k][m] = 0.0;
      if (!ok(k, m)) continue;
      const int c = cell(k, m);
      int i, j;
      cell_ij(c, nx, i, j);
      double b = MODE != 0 ? rhs_at(D, c, i, j, D.td ? t_sub(D, sub) : nullptr) : D.rhs[c];
      if (MODE == 2) {
        const LevelDev A = level(D, 0);
        const double *WX = D.wx, *WY = D.wy;
        const double wxc = WX[c], wyc = WY[c], xc = x[k][m];
        const double hdy = 0.5 * D.dy, hdx = 0.5 * D.dx;
        double corr = 0.0;
        if (i + 1 < nx) corr += A.ax[c] * (xc - X[c + 1]) + hdy * (wxc + WX[c + 1]);
        if (i > 0) corr += A.ax[c - 1] * (xc - X[c - 1]) - hdy * (wxc + WX[c - 1]);
        if (j + 1 < D.ny) corr += A.ay[c] * (xc - X[c + nx]) + hdx * (wyc + WY[c + nx]);
        if (j > 0) corr += A.ay[c - nx] * (xc - X[c - nx]) - hdx * (wyc + WY[c - nx]);
        b += corr;
      }
      if (MODE != 0) D.rhs[c] = b;
      r[k][m] = b - apply(k, m);
      rr = fma(r[k][m], r[k][m], rr);
      bb = fma(b, b, bb);
    }
  sum2(rr, bb);
  const double stop = fmax(D.rtol * D.rtol * rr, 1e-28 * bb);
  bool conv = !(rr > stop);
  int nit = 0;
  double ga_prev = 1.0, al_prev = 1.0;
  while (!conv && nit < max_it) {
    W.cycle();
    __syncthreads();
    double ga = 0.0, de = 0.0, w[2][M];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        w[k][m] = ok(k, m) ? apply(k, m) : 0.0;
        const double z = ok(k, m) ? *W.at(k, m) : 0.0;
        ga = fma(r[k][m], z, ga);
        de = fma(z, w[k][m], de);
      }
    sum2(ga, de);
    const CGCoef q = cg_coef(nit == 0, ga, de, ga_prev, al_prev);
    rr = 0.0;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const double z = ok(k, m) ? *W.at(k, m) : 0.0;
        p[k][m] = nit > 0 ? fma(q.be, p[k][m], z) : z;
        s[k][m] = nit > 0 ? fma(q.be, s[k][m], w[k][m]) : w[k][m];
        x[k][m] = fma(q.al, p[k][m], x[k][m]);
        r[k][m] = fma(-q.al, s[k][m], r[k][m]);
        rr = fma(r[k][m], r[k][m], rr);
      }
    double none = 0.0;
    sum2(rr, none);
    ga_prev = ga;
    al_prev = q.al;
    ++nit;
    conv = !(rr > stop);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (ok(k, m)) xg[cell(k, m)] = x[k][m];
  if (threadIdx.x == 0) {
    D.scal[S_NIT] = nit;
    D.state[3] = conv ? 1 + nit : 0;
  }
}

// ------------------------------------------------------------- update / Err
// delta = phi' - phi_half (GSIS) or 0 (SI); Err partials; phi = phi_new.
// FP32-mixed mode also records base = phi^m + delta (see the transport file).
// cond: launched ahead of the host's look at the synthetic solve's flags;
// runs only if that solve has converged (state[3]), else returns.
// state[5] tells the launch that follows (k_err_source) whether it ran: that
// launch's own end of the iteration changes state[1] while its source tiles run
__global__ void k_update(const SynthDesc *ds, const int2 *bt, int cond) {
  __shared__ double sh[kRedBlock];
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1] | (cond && D.state[3] == 0);   // tested after the operand loads
  const int c = B.lb * kRedBlock + threadIdx.x;
  const bool in = c < D.N;
  const int cc = in ? c : 0;
  const double pn = D.method ? D.lev[0].x[cc] : D.phih[cc];
  const double ph = D.phih[cc], po = D.phi[cc];
  // time-dependent form: T^{m+1} = T(sub_iter), against T^m for Err(T)
  const double tn = D.td ? t_sub(D, D.sub_iter)[cc] : 0.0, to = D.td ? D.Tm[cc] : 0.0;
  if (B.lb == 0 && threadIdx.x == 0) D.state[5] = f1 == 0;
  if (f1 != 0) return;
  double num = 0.0, den = 0.0, numT = 0.0, denT = 0.0;
  if (in) {
    const double d = pn - po;
    num = D.V * d * d;
    den = D.V * pn * pn;
    const double dl = D.method ? pn - ph : 0.0;
    D.delta[c] = dl;
    if (D.fp32) D.base[c] = po + dl;
    D.phi[c] = pn;
    if (D.td) {
      numT = D.V * (tn - to) * (tn - to);
      denT = D.V * tn * tn;
      D.Tm[c] = tn;
    }
  }
  double a = block_sum(num, sh);
  double b = block_sum(den, sh);
  if (threadIdx.x == 0) { D.err_parts[2 * B.lb] = a; D.err_parts[2 * B.lb + 1] = b; }
  if (D.td) {
    a = block_sum(numT, sh);
    b = block_sum(denT, sh);
    if (threadIdx.x == 0) { D.err_parts_T[2 * B.lb] = a; D.err_parts_T[2 * B.lb + 1] = b; }
  }
}

// SI in FP64, one problem: the moments' combine (f = blockIdx.y: phi, Fx, Fy
// from ns partials per quadrant, each quadrant's in order, then the quadrants)
// and, with phi, the update of k_update. As two kernels they were two launches
// of 5.0 and 4.9 us (40 x 40 x 1728); as one 5.8. (FP32-mixed sums need phi^m,
// which another block would be replacing.)
__global__ void k_update_combine(const SynthDesc *ds, int ns) {
  __shared__ double sh[2 * kRedBlock / 64];
  CDesc &D = cdesc(ds, 0);
  const int32_t f1 = D.state[1];   // tested after the loads
  const int c = blockIdx.x * kRedBlock + threadIdx.x, f = blockIdx.y;
  const bool in = c < D.N;
  const size_t N = D.N, cc = in ? c : 0;
  const double *p = D.mom_part + f * N + cc;
  const double po = D.phi[cc];
  double v[4] = {};
  int z = 0;
  for (; z + 4 <= ns; z += 4) {
    double u[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) u[m][q] = p[(12 * (size_t)(z + m) + 3 * q) * N];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += u[m][q];
  }
  for (; z < ns; ++z)
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] += p[(12 * (size_t)z + 3 * q) * N];
  if (blockIdx.x == 0 && f == 0 && threadIdx.x == 0) D.state[5] = f1 == 0;
  if (f1 != 0) return;
  double s = 0.0;
  for (int q = 0; q < 4; ++q) s += v[q];
  if (f > 0) {
    if (in) (f == 1 ? D.Fx : D.Fy)[c] = s;
    return;
  }
  double num = 0.0, den = 0.0;
  if (in) {
    const double d = s - po;
    num = D.V * d * d;
    den = D.V * s * s;
    D.phih[c] = s;
    D.delta[c] = 0.0;
    D.phi[c] = s;
  }
  block_sum2(num, den, sh);
  if (threadIdx.x == 0) {
    D.err_parts[2 * blockIdx.x] = num;
    D.err_parts[2 * blockIdx.x + 1] = den;
  }
}

// Time-dependent form: one step of the material equation per cell (Eqs.
// MSE_d2, R2_def, MSE_d_mtx2, elem_mtx_M),
//   T(sub + 1) = T(sub) + R2 / D2,
//   R2 = -cv (T(sub) - T^n) / dt + sigma_a (rho(sub) - a c T(sub)^4),
//   D2 = cv / dt + 4 a c T(sub)^3 sigma_a,
// with rho(sub) = rho^{m+1/2} for sub 0 and for source iteration, else the
// synthetic solution of sub-iteration sub - 1 (the level-0 iterate).
__global__ void k_material(const SynthDesc *ds, const int2 *bt, int sub) {
  const Blk B = blk(bt);
  CDesc &D = cdesc(ds, B.p);
  const int32_t f1 = D.state[1];
  const int c = B.lb * kRedBlock + threadIdx.x;
  if (c >= D.N) return;
  const double *Ts = t_sub(D, sub);
  double *To = ((sub & 1) ? D.Tsub1 : D.Tsub0);
  const double rho = (sub == 0 || !D.method) ? D.phih[c] : D.lev[0].x[c];
  const double T = Ts[c], T2 = T * T, sa = D.sig_a[c], cv = D.cv[c], dt = D.dt;
  const double R2 = -cv * (T - D.Tn[c]) / dt + sa * (rho - D.ca * (T2 * T2));
  const double D2 = cv / dt + 4.0 * D.ca * (T2 * T) * sa;
  if (f1 != 0) return;
  To[c] = T + R2 / D2;
}

// p[e t], p[e (t + blockDim)], ... (t = threadIdx.x; n terms in all) added
// in that order, the first loaded by the caller (that of every array before any
// is waited for); sixteen loads in flight at a time (terms past n add 0,
// and every sum here is of squares)
__device__ inline double strided_sum(const double *p, int n, int e, double first) {
  constexpr int U = 16;
  double s = (int)threadIdx.x < n ? first : 0.0;
  for (int t0 = threadIdx.x + blockDim.x; t0 < n; t0 += U * (int)blockDim.x) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * (int)blockDim.x;
      v[u] = t < n ? p[(size_t)e * t] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s += v[u];
  }
  return s;
}

// One workgroup per problem: Err = sqrt(num/den) -> history, counters, done
// flag; the relative transport residual of the iterate this iteration
// started from, sqrt(sum w r^2 / (sum_k w_k sum_c src^2)) (the cell volume
// cancels on a uniform grid), from the residual kernel's per-wave partials
// and the moments kernel's per-block partials of the same iteration.
// Divergence: Err not finite, or the change ||phi^{m+1} - phi^m||_V above
// 1e3 times its smallest value so far (floored at 1e-9 ||phi^{m+1}||_V, far
// above rounding); Err alone cannot show a geometric blow-up, it tends to
// |1 - 1/g| for a growth factor g. last_err[1] keeps that smallest change.
__device__ inline void err_finish(CDesc &D, double *sh) {
  int32_t *state = D.state;
  const int npart = nblk_d(D.N);
  // the first partials and the scalars before the flag is tested
  auto first = [](const double *p, int n, int e) {
    return p[(int)threadIdx.x < n ? (size_t)e * threadIdx.x : 0];
  };
  const double *pe = D.err_parts, *pt = D.td ? D.err_parts_T : pe;
  const double a0 = first(pe, npart, 2), b0 = first(pe + 1, npart, 2);
  const double r0 = first(D.tres_part, D.n_tres, 1), q0 = first(D.src2_part, D.n_src2, 1);
  const double s0 = first(pt, npart, 2), t0 = first(pt + 1, npart, 2);
  if (state[1] != 0) return;
  // (the residual-norm partials number one per residual wave: tens of
  // thousands on large grids)
  double a = strided_sum(pe, npart, 2, a0), b = strided_sum(pe + 1, npart, 2, b0);
  double rr = strided_sum(D.tres_part, D.n_tres, 1, r0);
  double ss = strided_sum(D.src2_part, D.n_src2, 1, q0);
  double aT = 0.0, bT = 0.0;
  if (D.td) {
    aT = strided_sum(pt, npart, 2, s0);
    bT = strided_sum(pt + 1, npart, 2, t0);
  }
  const double dmin = D.last_err[1];
  // the sums side by side: wave sums, then in wave order
  double sums[6] = {a, b, rr, ss, aT, bT};
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    if (e >= 4 && !D.td) break;
    const double w = wave_sum(sums[e]);
    if ((threadIdx.x & 63) == 0) sh[6 * (threadIdx.x >> 6) + e] = w;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    if (e >= 4 && !D.td) break;
    sums[e] = 0.0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) sums[e] += sh[6 * k + e];
  }
  const double num = sums[0], den = sums[1];
  rr = sums[2];
  ss = sums[3] * D.sw;
  aT = sums[4];
  bT = sums[5];
  double err = den > 0.0 ? sqrt(num / den) : (num == 0.0 ? 0.0 : INFINITY);
  if (D.td) {    // max(Err(rho), Err(T)), the criterion after Eq. Err_W
    const double eT = bT > 0.0 ? sqrt(aT / bT) : (aT == 0.0 ? 0.0 : INFINITY);
    err = eT > err ? eT : err;
  }
  const double tres = ss > 0.0 ? sqrt(rr / ss) : (rr == 0.0 ? 0.0 : INFINITY);
  const int m = state[0];
  D.err_hist[m] = err;
  D.tres_hist[m] = tres;
  // V-cycles of this iteration's (last) synthetic solve: the first after
  // the warm start, one per CG iteration
  if (D.method) D.scal[S_VCYCLES] += D.scal[S_NIT] + 1.0;
  const double dn = sqrt(num), pn = sqrt(den);
  D.last_err[0] = err;
  if (dn < dmin) D.last_err[1] = dn;
  state[0] = m + 1;
  state[2] = 1 - state[2];   // I^{m+1} now lives in the other buffer
  if (!isfinite(err) || dn > 1e3 * fmax(dmin, 1e-9 * pn)) state[1] = -1;
  else if (err < D.tol) state[1] = 1;
  else if (m + 1 >= D.max_iter) state[1] = 2;
}

// src = (sigma_s phi + q) / (4 pi); the mirrored per-quadrant copies of
// (src, base/(4 pi), phi/(4 pi)) read by the transport kernels, stored in
// each quadrant's anti-diagonal order. One workgroup per 16 x 16 tile: the
// values go through LDS, then for every quadrant thread t writes the tile's
// t-th cell in that quadrant's anti-diagonal order, so the cells of a
// diagonal run over consecutive lanes and consecutive addresses.
constexpr int kSrcT = 16;
static_assert(kSrcT * kSrcT == kRedBlock, "one thread per tile cell");
// run: 0 leaves the source as it is.
__device__ inline void source_tile(CDesc &D, const Blk &B, double *s_sc, double *s_dq,
                                   double *s_pq, const int32_t run) {
  const int nx = D.nx, ny = D.ny, n = D.N;
  int ti, tj;
  cell_ij(B.lb, (nx + kSrcT - 1) / kSrcT, ti, tj);
  const int i0 = ti * kSrcT, j0 = tj * kSrcT;
  const int t = threadIdx.x;
  {
    const int i = i0 + (t & (kSrcT - 1)), j = j0 + t / kSrcT;
    const bool in = i < nx && j < ny;
    const int c = in ? j * nx + i : 0;
    double sc = (D.sig_s[c] * D.phi[c] + D.q[c]) / kFourPi;
    if (D.td) {                  // emission sigma_a a c (T^m)^4 / (4 pi)
      const double T = D.Tm[c], T2 = T * T;
      sc = (D.sig_s[c] * D.phi[c] + D.sig_a[c] * (D.ca * (T2 * T2)) + D.q[c]) / kFourPi;
    }
    const double dq = D.base[c] / kFourPi;
    const double pq = D.phi[c] / kFourPi;
    if (run == 0) return;          // (tested after the operands are loaded)
    if (in) D.src[c] = sc;
    s_sc[t] = sc; s_dq[t] = dq; s_pq[t] = pq;
  }
  __syncthreads();
  int u, w;                      // cell t of the square in anti-diagonal order
  square_diag<kSrcT>(t, u, w);
  for (int qd = 0; qd < 4; ++qd) {
    // the square in quadrant qd's mirrored frame: u runs against x when x
    // is mirrored, w against y when y is
    const int i = (qd & 1) ? i0 + kSrcT - 1 - u : i0 + u;
    const int j = (qd & 2) ? j0 + kSrcT - 1 - w : j0 + w;
    if (i >= nx || j >= ny) continue;
    const int xl = (qd & 1) ? nx - 1 - i : i, yl = (qd & 2) ? ny - 1 - j : j;
    const size_t o = (size_t)qd * 3 * n + dg_idx(xl, yl, nx, ny);
    const int l = (j - j0) * kSrcT + (i - i0);
    D.dynq[o] = s_sc[l];          // plane 0 of quadrant qd
    D.dynq[o + n] = s_dq[l];      // plane 1
    if (D.fp32) D.dynq[o + 2 * n] = s_pq[l];
  }
}

__global__ void __launch_bounds__(kRedBlock) k_source(const SynthDesc *ds, const int2 *bt) {
  __shared__ double s_sc[kRedBlock], s_dq[kRedBlock], s_pq[kRedBlock];
  const Blk B = blk(bt);
  source_tile(cdesc(ds, B.p), B, s_sc, s_dq, s_pq, 1);
}

// End of an outer iteration: blocks [0, n) finish Err of problem blockIdx.x,
// blocks from n8 (n rounded up to a multiple of 8) make source tiles (table
// bt, or one problem's tiles). The two do not depend on each other: the
// source is written also on the iteration that ends the solve (a
// time-dependent step starts from it), so its tiles go by state[5], which
// k_update left, not by state[1], which the blocks before them may be setting
// (from some 2000 tiles on, the last ones start after that). One problem:
// its ntile tiles (row-major) fall into 8 runs of ts, one per XCD (block
// n8 + b runs on XCD b % 8 and takes tile (b % 8) ts + b / 8), so the
// partly written cache lines at the ends of a tile's diagonal runs mostly
// meet the neighbouring tile's part in the same L2.
// Latency is all of it on small grids: the first partials of every sum are
// loaded together, the sums are reduced side by side, a thread finds its place
// on the diagonals in closed form. 32 x 32: 5.5 to 3.7 us, 40 x 40 with 1728
// ordinates 5.8 to 4.8, 128 x 128 (time-dependent) 7.3 to 6.0.
__global__ void __launch_bounds__(kRedBlock) k_err_source(const SynthDesc *ds, const int2 *bt,
                                                          int n, int n8, int ntile, int ts,
                                                          int cond) {
  __shared__ double s_sc[kRedBlock], s_dq[kRedBlock], s_pq[kRedBlock];
  if ((int)blockIdx.x < n) {
    CDesc &D = cdesc(ds, blockIdx.x);
    if (cond && D.state[3] == 0) return;   // as k_update
    err_finish(D, s_sc);
    return;
  }
  const int idx = blockIdx.x - n8;
  if (idx < 0) return;
  Blk B;
  if (bt) {
    const __attribute__((address_space(4))) int *q =
        (const __attribute__((address_space(4))) int *)bt;
    B = {q[2 * idx], q[2 * idx + 1]};
  } else {
    const int tile = (idx & 7) * ts + (idx >> 3);
    if (tile >= ntile || (idx >> 3) >= ts) return;
    B = {0, tile};
  }
  CDesc &D = cdesc(ds, B.p);
  if (cond && D.state[3] == 0) return;
  source_tile(D, B, s_sc, s_dq, s_pq, D.state[5]);
}

// z = M^{-1} r_v (one V(1,1) cycle with scaled coarse corrections) for
// every problem of the set, with the partials of r.z. V-cycle v > 0 follows
// CG iteration v - 1, whose update its level-0 tile kernel makes. part 1
// launches only that level-0 kernel, part 2 the rest, after k_rr_test has
// made the r.r test (problems that start with a tile level); part 0 all.
void vcycle(const SynthSet &S, int v, hipStream_t s, int part = 0) {
  const SynthDesc *ds = S.desc;
  const int rr_ext = part == 2 ? 1 : 0;
  for (int l = part == 2 ? 1 : 0; l < (part == 1 ? 1 : S.max_lc); ++l)
    hipLaunchKernelGGL(k_mg_down, dim3(S.nb_tile[l]), dim3(kRedBlock), 0, s, ds, S.bt_tile[l], l,
                       v, rr_ext);
  if (part == 1) return;
  const dim3 gw(S.n), bw(kCoarseThreads);
  auto coarse = [&](auto m, auto sums) {
    hipLaunchKernelGGL((k_mg_coarse<decltype(m)::value, decltype(sums)::value>), gw, bw,
                       S.coarse_lds, s, ds, kOmega, v, rr_ext);
  };
  auto by_cells = [&](auto sums) {
    if (S.coarse_cells <= 2 * kCoarseThreads) coarse(std::integral_constant<int, 1>(), sums);
    else if (S.coarse_cells <= 4 * kCoarseThreads) coarse(std::integral_constant<int, 2>(), sums);
    else if (S.coarse_cells <= 6 * kCoarseThreads) coarse(std::integral_constant<int, 3>(), sums);
    else coarse(std::integral_constant<int, 4>(), sums);
  };
  if (S.any_sums) by_cells(std::true_type());
  else by_cells(std::false_type());
  for (int l = S.max_lc - 1; l >= 1; --l)
    hipLaunchKernelGGL(k_mg_up, dim3(S.nb_tile[l]), dim3(kRedBlock), 0, s, ds, S.bt_tile[l], l, v,
                       kOmega);
  if (S.max_lc > 0)
    hipLaunchKernelGGL(k_mg_up0, dim3(S.nb_tile[0]), dim3(kRedBlock), 0, s, ds, S.bt_tile[0], v,
                       kOmega);
  if (S.any_zw)
    hipLaunchKernelGGL(k_cg_zw, dim3(S.nb_cell), dim3(kRedBlock), 0, s, ds, S.bt_cell, v);
  if (S.any_coef_sep)
    hipLaunchKernelGGL(k_cg_coef, dim3(S.n), dim3(kRedBlock), 0, s, ds, v);
}

}  // namespace

// ------------------------------------------------------------ host side
size_t coarse_lds_bytes_from(const PlanDev &P, size_t lc) {
  size_t n = coarse_top_words(P.mg[lc].nx, P.mg[lc].ny, lc + 1 == P.mg.size());
  for (size_t l = lc + 1; l < P.mg.size(); ++l) n += 7 * (size_t)P.mg[l].nx * P.mg[l].ny;
  return n * sizeof(double);
}

// First level handled by the single-workgroup kernel: at most kCoarseCells
// cells and its vectors plus the lower levels' operators within the LDS budget
// (160 KB per CU, some of it static in the kernels).
constexpr size_t kCoarseLdsBudget = 156 * 1024;
int coarse_start(const PlanDev &P) {
  int lc = 0;
  while (lc + 1 < (int)P.mg.size() &&
         (P.mg[lc].nx * P.mg[lc].ny > kCoarseCells || coarse_lds_bytes_from(P, lc) > kCoarseLdsBudget))
    ++lc;
  return lc;
}

size_t coarse_lds_bytes(const PlanDev &P) { return coarse_lds_bytes_from(P, coarse_start(P)); }

int tiles_of(int nx, int ny) { return ((nx + kTW - 1) / kTW) * ((ny + kTH - 1) / kTH); }
int source_tiles_of(int nx, int ny) {
  return ((nx + kSrcT - 1) / kSrcT) * ((ny + kSrcT - 1) / kSrcT);
}

int coarse_cells(const PlanDev &P) {
  const MGLevel &L = P.mg[coarse_start(P)];
  return L.nx * L.ny;
}

// The attribute is per kernel, not per plan: it is raised to the largest
// amount any plan may ask for, so that a later plan with a smaller coarse
// cycle never lowers it under an earlier one.
void prepare_synth(size_t coarse_lds) {
  if (coarse_lds <= 64 * 1024) return;
  const void *ks[] = {(const void *)&k_mg_coarse<1, false>, (const void *)&k_mg_coarse<2, false>,
                      (const void *)&k_mg_coarse<3, false>, (const void *)&k_mg_coarse<4, false>,
                      (const void *)&k_mg_coarse<1, true>,  (const void *)&k_mg_coarse<2, true>,
                      (const void *)&k_mg_coarse<3, true>,  (const void *)&k_mg_coarse<4, true>,
                      (const void *)&k_cg_small<1, 0>, (const void *)&k_cg_small<1, 1>,
                      (const void *)&k_cg_small<1, 2>, (const void *)&k_cg_small<1, 3>,
                      (const void *)&k_cg_small<2, 0>, (const void *)&k_cg_small<2, 1>,
                      (const void *)&k_cg_small<2, 2>, (const void *)&k_cg_small<2, 3>,
                      (const void *)&k_cg_small<3, 0>, (const void *)&k_cg_small<3, 1>,
                      (const void *)&k_cg_small<3, 2>, (const void *)&k_cg_small<3, 3>,
                      (const void *)&k_cg_small<4, 0>, (const void *)&k_cg_small<4, 1>,
                      (const void *)&k_cg_small<4, 2>, (const void *)&k_cg_small<4, 3>};
  for (const void *k : ks)
    (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCoarseLdsBudget);
}

SynthDesc make_synth_desc(const PlanDev &P) {
  SynthDesc D;
  memset(&D, 0, sizeof D);
  D.nx = P.nx; D.ny = P.ny; D.N = P.N;
  D.dx = P.dx; D.dy = P.dy; D.V = P.V;
  D.method = P.method; D.fp32 = P.precision == GSIS_FP32_MIXED ? 1 : 0; D.max_iter = P.max_iter;
  D.tol = P.tol; D.rtol = P.synth_rtol;
  D.sig_t = P.sig_t; D.sig_s = P.sig_s; D.q = P.q;
  D.cE = P.cE; D.cW = P.cW; D.cN = P.cN; D.cS = P.cS; D.kappa = P.kappa;
  D.phih = P.phih; D.Fx = P.Fx; D.Fy = P.Fy; D.bflux = P.bflux;
  D.mom_part = P.mom_part; D.sw = P.sw; D.swm = P.swm; D.swe = P.swe;
  D.hot_face = P.method == GSIS_GSIS ? P.hot_face : 0;
  D.ftp = P.ftp;
  D.sig_a = P.sig_a;
  D.td = P.td; D.sub_iter = P.sub_iter; D.tdiag = P.tdiag; D.ca = P.ca; D.dt = P.dt;
  D.cv = P.cv; D.Tn = P.Tn; D.rho_n = P.rho_n; D.Tm = P.Tm; D.Tsub0 = P.Tsub0;
  D.Tsub1 = P.Tsub1; D.err_parts_T = P.err_parts_T;
  D.hx = P.hx; D.hy = P.hy; D.rhs = P.rhs; D.phi = P.phi; D.delta = P.delta; D.base = P.base;
  D.src = P.src; D.dynq = P.dynq;
  D.cg_r = P.cg_r; D.cg_r2 = P.cg_r2; D.cg_z = P.cg_z; D.cg_p = P.cg_p;
  D.cg_s0 = P.cg_s0; D.cg_s1 = P.cg_s1; D.cg_w = P.cg_w;
  D.wx = P.wide_wx; D.wy = P.wide_wy;
  D.red = P.red; D.scal = P.scal; D.err_parts = P.err_parts; D.err_hist = P.err_hist;
  D.last_err = P.last_err; D.state = P.state;
  D.tres_part = P.tres_part; D.src2_part = P.src2_part; D.tres_hist = P.tres_hist;
  D.n_tres = P.n_tres;
  D.n_src2 = nblk(P.N);
  D.nlev = (int)P.mg.size();
  for (int l = 0; l < D.nlev && l < kMaxLevels; ++l) {
    const MGLevel &L = P.mg[l];
    D.lev[l] = LevelDev{L.nx, L.ny, L.fx, L.fy, L.diag, L.ax, L.ay, L.x, L.b, L.r};
  }
  const int lc = coarse_start(P);
  D.lc = lc;
  D.ntile0 = tiles_of(P.mg[0].nx, P.mg[0].ny);
  D.ntp = std::max(D.ntile0, nblk(P.N));
  D.coef_sep = lc == 0 ? (D.fp32 ? 0 : kCoefCoarse)
                       : D.ntile0 >= kCoefSepTiles ? kCoefKernel : 0;
  // the record of the one-workgroup kernels
  int32_t *w = D.cl.w;
  auto ptr = [&](int k, const void *p) { memcpy(w + k, &p, sizeof p); };
  const int nlev = D.nlev - lc;
  w[kCwLast] = nlev - 1;
  w[kCwLc] = lc;
  w[kCwNb] = nblk(P.N);
  w[kCwTile] = D.ntile0;
  w[kCwRrt] = 2 * nblk(P.N) + D.ntp;   // red_rrt
  ptr(kCwRed, P.red);
  ptr(kCwScal, P.scal);
  ptr(kCwB0, lc == 0 ? P.cg_r : P.mg[lc].b);
  ptr(kCwB1, lc == 0 ? P.cg_r2 : P.mg[lc].b);
  ptr(kCwX, lc == 0 ? P.cg_z : P.mg[lc].x);
  ptr(kCwInv, P.coarse_inv);
  memcpy(w + kCwRtol, &D.rtol, sizeof D.rtol);
  w[kCwSums] = D.coef_sep == kCoefCoarse ? 1 : 0;
  int off = 0;
  for (int t = 0; t < nlev; ++t) {
    const MGLevel &L = P.mg[lc + t];
    const int n = L.nx * L.ny;
    int32_t *r = w + kCwLev + 4 * t;
    r[0] = L.nx | L.ny << 16;
    r[1] = off | (t + 1 < nlev && L.fx == 2 ? 1 << 20 : 0) | (t + 1 < nlev && L.fy == 2 ? 1 << 21 : 0);
    ptr(kCwLev + 4 * t + 2, L.diag);   // ay and ax follow
    off += t == 0 ? coarse_top_words(L.nx, L.ny, nlev == 1) : 7 * n;
  }
  return D;
}

void launch_source(const SynthSet &S, hipStream_t s) {
  hipLaunchKernelGGL(k_source, dim3(S.nb_src), dim3(kRedBlock), 0, s, S.desc, S.bt_src);
}

void launch_wide_grad(const SynthSet &S, hipStream_t s, bool first) {
  if (first)
    hipLaunchKernelGGL(k_wide_grad<true>, dim3(S.nb_cell), dim3(kRedBlock), 0, s, S.desc, S.bt_cell);
  else
    hipLaunchKernelGGL(k_wide_grad<false>, dim3(S.nb_cell), dim3(kRedBlock), 0, s, S.desc, S.bt_cell);
}

void launch_hot(const SynthSet &S, hipStream_t s, bool combine) {
  if (combine)
    hipLaunchKernelGGL(k_hot<true>, dim3(S.nb_cell), dim3(kRedBlock), 0, s, S.desc, S.bt_cell);
  else
    hipLaunchKernelGGL(k_hot<false>, dim3(S.nb_cell), dim3(kRedBlock), 0, s, S.desc, S.bt_cell);
}

// Preconditioned CG (the Chronopoulos-Gear form, see cg_coef) on D1 phi' =
// rhs for every problem of the set, each warm-started from its phi (the
// previous synthetic solution), preconditioned by one V-cycle per
// iteration; solutions land in level 0's x. An iteration is one V-cycle:
// its level-0 down kernel makes the previous iteration's update, its
// level-0 up kernel forms w = A z and the partials of r.z and z.w, and
// every reduction is finished inside the kernel that needs it (see the
// partial regions above). The stop test runs on the device (state[3] per
// problem: 1 + the iterations taken once converged). With host_flag (a
// single problem), the host stops launching once the solve has converged:
// it checks the device flags after the V-cycle that would make the test at
// the iteration count the previous solve took (host_flag[8] keeps that
// count) and after every later one, so a run whose counts stay level waits
// once per solve and launches no V-cycle past convergence. Without it
// (batches, graph capture) exactly synth_max_iter iterations are launched
// and converged problems skip their kernels. spec (an event; single plans,
// plain GSIS): at each check the end of the outer iteration (launch_update,
// made conditional on convergence) is put into the stream before the host
// waits; true is returned when the solve has converged at a check, the
// update then being in the stream.
// FP64 sets whose every problem starts with the one-workgroup cycle run the
// whole solve in one kernel (k_cg_small) and never wait. Its sums of products
// are added by cell owners; beside larger problems the coarse cycle forms them
// so (kCoefCoarse: the r.r test, w = A z and the CG coefficients), where other
// problems of that size have k_cg_zw and block partials. An FP32-mixed step
// rounds differences of the iterate to floats, which turns one unit in the last
// place of phi into 1e-8 of the flux, so those plans keep the block partials'
// order. (The small problems' whole solves after or beside the others': 10
// iterations of 16 problems 5.6 and 5.1 ms, of 6 3.19 and 3.44; with the sums in
// the coarse cycle 5.1 and 3.0, with block partials, k_cg_zw among the launches,
// 5.1 and 3.1.)
namespace {
template <int M>
void launch_cg_small(const SynthSet &S, hipStream_t s, int rhs_mode, int sub) {
  const dim3 g(S.n), b(kCoarseThreads);
  const int mi = S.synth_max_iter;
  if (rhs_mode == 1) hipLaunchKernelGGL((k_cg_small<M, 1>), g, b, S.coarse_lds, s, S.desc, sub, mi);
  else if (rhs_mode == 2) hipLaunchKernelGGL((k_cg_small<M, 2>), g, b, S.coarse_lds, s, S.desc, sub, mi);
  else if (rhs_mode == 3) hipLaunchKernelGGL((k_cg_small<M, 3>), g, b, S.coarse_lds, s, S.desc, sub, mi);
  else hipLaunchKernelGGL((k_cg_small<M, 0>), g, b, S.coarse_lds, s, S.desc, sub, mi);
}
}  // namespace
bool launch_synth_solve(const SynthSet &S, hipStream_t s, int32_t *host_flag, int rhs_mode,
                        int sub, hipEvent_t spec) {
  const SynthDesc *ds = S.desc;
  if (synth_in_one_kernel(S)) {
    if (S.coarse_cells <= 2 * kCoarseThreads) launch_cg_small<1>(S, s, rhs_mode, sub);
    else if (S.coarse_cells <= 4 * kCoarseThreads) launch_cg_small<2>(S, s, rhs_mode, sub);
    else if (S.coarse_cells <= 6 * kCoarseThreads) launch_cg_small<3>(S, s, rhs_mode, sub);
    else launch_cg_small<4>(S, s, rhs_mode, sub);
    return false;
  }
  const dim3 gc(S.nb_cell), bk(kRedBlock);
  if (rhs_mode == 1) hipLaunchKernelGGL(k_cg_begin<1>, gc, bk, 0, s, ds, S.bt_cell, sub);
  else if (rhs_mode == 2) hipLaunchKernelGGL(k_cg_begin<2>, gc, bk, 0, s, ds, S.bt_cell, sub);
  else if (rhs_mode == 3) hipLaunchKernelGGL(k_cg_begin<3>, gc, bk, 0, s, ds, S.bt_cell, sub);
  else hipLaunchKernelGGL(k_cg_begin<0>, gc, bk, 0, s, ds, S.bt_cell, sub);
  vcycle(S, 0, s);
  const int guess = host_flag ? host_flag[8] : 0;
  for (int it = 0; it < S.synth_max_iter; ++it) {
    if (it + 1 == S.synth_max_iter) {
      // no V-cycle follows: the update on its own, then the r.r test
      hipLaunchKernelGGL(k_cg_update, gc, bk, 0, s, ds, S.bt_cell, it, 1);
      hipLaunchKernelGGL(k_finish_rr, dim3(S.n), bk, 0, s, ds);
      break;
    }
    // problems whose V-cycle runs wholly in the one-workgroup kernel have
    // no level-0 tile kernel to make the update
    if (S.min_lc == 0) hipLaunchKernelGGL(k_cg_update, gc, bk, 0, s, ds, S.bt_cell, it, 0);
    const bool due = guess > 0 ? it + 1 >= guess : (it >= 3 && ((it - 3) & 1) == 0);
    const bool check = host_flag && S.state0 && due;
    // at a check of a problem that starts with a tile level, the update and
    // the r.r test go first and the rest of the V-cycle only if it fails
    const bool split = check && S.n == 1 && S.min_lc >= 1;
    if (split) {
      vcycle(S, it + 1, s, 1);   // the update (level 0)
      hipLaunchKernelGGL(k_rr_test, dim3(S.n), bk, 0, s, ds);
    } else {
      vcycle(S, it + 1, s);   // makes the update (level 0) and the r.r test
    }
    if (check) {
      (void)hipMemcpyAsync(host_flag, S.state0 + 1, 3 * sizeof(int32_t), hipMemcpyDeviceToHost,
                           s);
      if (spec) {
        // the end of the outer iteration goes into the stream before the
        // host waits (on the flags' copy alone); it runs only if the solve
        // has converged, so the GPU need not idle while the host wakes
        (void)hipEventRecord(spec, s);
        launch_update(S, s, 1);
        (void)hipEventSynchronize(spec);
      } else {
        (void)hipStreamSynchronize(s);
      }
      if (host_flag[0] != 0) return false;
      if (host_flag[2] != 0) {
        host_flag[8] = max(1, host_flag[2] - 1);
        return spec != nullptr;
      }
      if (split) vcycle(S, it + 1, s, 2);
    }
  }
  return false;
}

void launch_material(const SynthSet &S, hipStream_t s, int sub) {
  hipLaunchKernelGGL(k_material, dim3(S.nb_cell), dim3(kRedBlock), 0, s, S.desc, S.bt_cell, sub);
}

void launch_update(const SynthSet &S, hipStream_t s, int cond, int combine) {
  if (combine)
    hipLaunchKernelGGL(k_update_combine, dim3(S.nb_cell, 3), dim3(kRedBlock), 0, s, S.desc, combine);
  else
    hipLaunchKernelGGL(k_update, dim3(S.nb_cell), dim3(kRedBlock), 0, s, S.desc, S.bt_cell, cond);
  const int n8 = (S.n + 7) / 8 * 8, ts = (S.nb_src + 7) / 8;
  const int nb = S.bt_src ? S.nb_src : 8 * ts;
  hipLaunchKernelGGL(k_err_source, dim3(n8 + nb), dim3(kRedBlock), 0, s, S.desc, S.bt_src, S.n,
                     n8, S.nb_src, ts, cond);
}

double *synth_iteration_counter(const PlanDev &P) { return P.scal + S_NIT; }
double *synth_vcycle_total(const PlanDev &P) { return P.scal + S_VCYCLES; }

}  // namespace gsis
