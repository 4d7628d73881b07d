// Single-workgroup float64 solves on the p x p projected problem: the stop test and
// Polak-Ribiere coefficient, the eigendecomposition of P^T P (one-sided Jacobi on its
// Cholesky factor, warm-started from the previous iteration's eigenvectors), the line-search
// diagonals,
// the exact line search (bracket from the branch roots, Brent's method on phi'), the
// retraction factor M, Cholesky QR and Rayleigh-Ritz.
//
// The p x p matrices live in the small buffer as PP x PP row-major arrays (PP = 16, 32, 64 or
// 128, the smallest that holds p) whose padding is zero; dense products among them use f64
// MFMA. Working matrices sit in LDS up to PP = 64 and in the small buffer's work area above.
#include <math.h>

#include "gsi_kernels.h"
#include "gsi_small_dev.h"

namespace gsi {

// ---------------------------------------------------------------- kernels

// The reduction of a pass's partial sums (see k_reduce) by the single workgroup that consumes
// them, when there are few (FOLD_MAX): the reduction's launch is saved. Ends with a barrier.
__device__ __forceinline__ void fold_partials(const double* __restrict__ partials, int nb, int nv, int max_from,
                                              double* __restrict__ red) {
  for (int v = threadIdx.x; v < nv; v += blockDim.x) {
    const bool use_max = v >= max_from;
    double s = 0.0;
#pragma unroll 8
    for (int b = 0; b < nb; ++b) {
      const double x = partials[(int64_t)b * nv + v];
      s = use_max ? fmax(s, x) : s + x;
    }
    red[v] = s;
  }
  __syncthreads();
}

__global__ __launch_bounds__(WG) void k_after_grad(int PP, double* red, double* __restrict__ small,
                                                   Scalars* __restrict__ sc, double* __restrict__ hist, int cond,
                                                   Partials fold) {
  if (sc->done) return;
  if (cond == GRAD_PENDING && sc->grad_ready) return;
  if (cond >= GRAD_AFTER_FUSED && (sc->null_step || sc->refresh || sc->grad_ready)) {
    // the short sequence has no kernels for what comes next (the gradient's own pass, an
    // explicit A X): its remaining launches return at once and the host runs the full one
    if (cond == GRAD_AFTER_LEAN && threadIdx.x == 0) sc->done = DONE_HOLD;
    return;
  }
  if (fold.nb) fold_partials(fold.p, fold.nb, PP * PP + 3, PP * PP + 2, red);
  __shared__ double sbeta, sphi;
  // the scalars and the trace of C are read by all threads at once (one round trip) and the
  // sequential decisions below work on the LDS copy: dependent global reads one after the
  // other cost a memory latency each
  __shared__ Scalars ls;
  for (int i = threadIdx.x; i < (int)(sizeof(Scalars) / 4); i += blockDim.x)
    reinterpret_cast<int32_t*>(&ls)[i] = reinterpret_cast<const int32_t*>(sc)[i];
  if (threadIdx.x < 64) {
    double d = 0.0;
    for (int i = threadIdx.x; i < PP; i += 64) d += small[S_C * PP * PP + i * PP + i];
    d = wave_sum(d);
    if (threadIdx.x == 0) sphi = -0.5 * d;
  }
  __syncthreads();
  const double* K = red;
  if (threadIdx.x == 0) {
    Scalars* lsc = &ls;
    const double gg = red[PP * PP], gdot = red[PP * PP + 1], ginf = red[PP * PP + 2];
    const int k = lsc->k;
    sc->gg = gg;
    sc->gdot = gdot;
    sc->ginf = ginf;
    const double rho = sqrt(gg) / (lsc->sqrt_p * lsc->nA);
    const double phi = sphi;
    sc->rho = rho;
    sc->phi = phi;
    if (k == 0) {
      lsc->ginf0 = ginf;
      sc->ginf0 = ginf;
    }
    if (k < lsc->hist_cap) {
      double* h = hist + (int64_t)k * H_FIELDS;
      h[H_RHO] = rho;
      h[H_PHI] = phi;
      h[H_MU] = 0.0;
      h[H_BETA] = 0.0;
      h[H_GINF] = lsc->ginf0 > 0.0 ? ginf / lsc->ginf0 : 0.0;
      if (k + 1 > lsc->hist_len) sc->hist_len = k + 1;
    }
    double beta = 0.0;
    if (k == 0 || rho <= 0.5 * lsc->rho_best) {
      lsc->rho_best = rho;
      lsc->k_best = k;
      sc->rho_best = rho;
      sc->k_best = k;
    }
    if (!isfinite(gg)) {
      ls.done = sc->done = 3;
    } else if (rho <= lsc->tol) {
      ls.done = sc->done = 1;
    } else if (k >= lsc->max_iter) {
      ls.done = sc->done = 2;
    } else if (lsc->stall_window > 0 && k - lsc->k_best > lsc->stall_window) {
      ls.done = sc->done = 4;  // stagnation: the block precision cannot resolve further progress
    } else {
      const bool restart = lsc->method == 1 || k == 0 || lsc->restart_next ||
                           (lsc->k_restart > 0 && k % lsc->k_restart == 0) || !(lsc->gg_old > 0.0);
      beta = restart ? 0.0 : (gg - gdot) / lsc->gg_old;
      sc->restart = restart ? 1 : 0;
      sc->restart_next = 0;
      sc->null_step = 0;
      sc->beta_pr = beta;
      if (k < lsc->hist_cap) hist[(int64_t)k * H_FIELDS + H_BETA] = beta;
    }
    sbeta = beta;
    sc->grad_ready = 1;
  }
  __syncthreads();
  if (ls.done) return;
  const double beta = sbeta;
  double* Kd = small + S_KD * PP * PP;
  double* Ks = small + S_K * PP * PP;
  const double* W = small + S_W * PP * PP;
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
    Ks[e] = K[e];
    Kd[e] = K[e] + (beta != 0.0 ? beta * W[e] : 0.0);
  }
}

__global__ __launch_bounds__(WG) void k_after_dir(int PP, double* red, double* __restrict__ small,
                                                  Scalars* __restrict__ sc, Partials fold) {
  if (sc->done) return;
  if (fold.nb) fold_partials(fold.p, fold.nb, PP * PP + 1, PP * PP + 1, red);
  double* S = small + S_S * PP * PP;
  // lane j of each wave, rows dealt to the waves (no division by the runtime PP)
  for (int i = threadIdx.x >> 6; i < PP; i += blockDim.x >> 6)
    for (int j = threadIdx.x & 63; j < PP; j += 64) S[i * PP + j] = 0.5 * (red[i * PP + j] + red[j * PP + i]);
  if (threadIdx.x == 0) {
    const double gp = red[PP * PP];
    sc->gp = gp;
    if (!(gp > 0.0)) {
      if (sc->restart) {
        sc->done = 3;  // the projected gradient is not a descent direction: G = 0 to rounding
      } else {
        sc->null_step = 1;
        sc->restart_next = 1;
        sc->n_null += 1;
        sc->grad_ready = 0;  // the next iteration forms the gradient again (and restarts)
      }
    }
  }
}

// Eigendecomposition of P^T P (see eig_dev), one workgroup.
template <int PP>
__global__ __launch_bounds__(dense_threads(PP)) void k_eig(double* __restrict__ small, Scalars* __restrict__ sc) {
  if (sc->done || sc->null_step) return;
  // this single workgroup shares its CU with the SpMM running concurrently: raise its
  // waves' issue priority so the latency-bound rotation rounds are not starved
  __builtin_amdgcn_s_setprio(3);
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int sweeps = eig_dev<PP>(small, sc->p, sc->v_valid != 0, reinterpret_cast<double*>(lds_raw));
  if (threadIdx.x == 0) {
    sc->v_valid = 1;
    sc->sweeps = sweeps;
    sc->n_sweeps += sweeps;
  }
}

// Line search and retraction factor (see linesearch_dev), one workgroup; red holds the
// reduced Grams P^T A P, P^T A X of the SpMM.
template <int PP>
__global__ __launch_bounds__(dense_threads(PP)) void k_linesearch(double* red, double* __restrict__ small, Scalars* __restrict__ sc,
                                                   double* __restrict__ hist, int recompute_ax, int want_mc,
                                                   Partials fold) {
  if (sc->done || sc->null_step) return;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ Terms terms;
  __shared__ double smu, sbmax;
  __shared__ int sok, sevals;
  // the scalars read by the sequential tail, loaded by all threads at once
  __shared__ Scalars ls;
  for (int i = threadIdx.x; i < (int)(sizeof(Scalars) / 4); i += blockDim.x)
    reinterpret_cast<int32_t*>(&ls)[i] = reinterpret_cast<const int32_t*>(sc)[i];
  if (fold.nb) fold_partials(fold.p, fold.nb, 2 * PP * PP, 2 * PP * PP, red);
  __syncthreads();
  linesearch_dev<PP>(red, red + PP * PP, small, ls.p, reinterpret_cast<double*>(lds_raw), terms, &smu, &sok, &sevals,
                     &sbmax, want_mc != 0);
  if (threadIdx.x == 0) {
    sc->brent_evals = sevals;
    sc->grad_ready = 0;  // X changes (or the step is void and the next iteration restarts)
    if (!sok) {
      if (ls.restart) {
        sc->done = 3;
      } else {
        sc->null_step = 1;
        sc->restart_next = 1;
        sc->n_null = ls.n_null + 1;
      }
    } else {
      const int k = ls.k;
      const double mu = smu;
      const int refresh = (recompute_ax || mu * sqrt(sbmax) <= 1e3 * EPS) ? 1 : 0;
      sc->mu = mu;
      sc->refresh = refresh;
      if (k < ls.hist_cap) hist[(int64_t)k * H_FIELDS + H_MU] = mu;
      sc->n_restart = ls.n_restart + ls.restart;
      sc->n_refresh = ls.n_refresh + refresh;
      sc->n_spmm = ls.n_spmm + 1 + refresh;
      sc->gg_old = ls.gg;
      sc->k = k + 1;
    }
  }
}

__global__ __launch_bounds__(WG) void k_after_update_grams(int PP, const double* __restrict__ red,
                                                           double* __restrict__ small, Scalars* __restrict__ sc) {
  if (sc->done || sc->null_step) return;
  double* C = small + S_C * PP * PP;
  double* W = small + S_W * PP * PP;
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
    const int i = e / PP, j = e % PP;
    if (!sc->refresh) C[e] = 0.5 * (red[i * PP + j] + red[j * PP + i]);
    W[e] = red[PP * PP + e];
  }
}

// hold: the next iteration is a short one, which needs the current gradient.
__global__ __launch_bounds__(WG) void k_after_refresh(int PP, const double* __restrict__ red,
                                                      double* __restrict__ small, Scalars* __restrict__ sc, int hold) {
  if (sc->done) return;
  const bool formed = !sc->null_step && sc->refresh;
  __syncthreads();
  if (formed) {
    double* C = small + S_C * PP * PP;
    for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
      const int i = e / PP, j = e % PP;
      C[e] = 0.5 * (red[i * PP + j] + red[j * PP + i]);
    }
  }
  if (threadIdx.x == 0) {
    if (formed) sc->refresh = 0;
    if (hold && !sc->grad_ready) sc->done = DONE_HOLD;
  }
}

// Cholesky G = L L^T of the leading p x p block of red, then M = L^{-T} (so X M has
// orthonormal columns when G = X^T X). flag = 1 on a non-positive or tiny pivot.
template <int PP>
__global__ __launch_bounds__(dense_threads(PP)) void k_chol_inv(int p, const double* __restrict__ red,
                                                                double* __restrict__ small, int* __restrict__ flag) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr int LD = DLD<PP>;
  constexpr bool wide = PP > PP_LDS_MAX;  // L alone fits LDS then
  double* A = reinterpret_cast<double*>(lds_raw);
  double* Mb = wide ? small + small_work_offset(PP) + 4 * PP * (PP + 1) : A + PP * LD;
  const int m = 16 * ((p + 15) >> 4), l = threadIdx.x & 63;
  double dmax = 0.0;
  for (int i = l; i < p; i += 64) dmax = fmax(dmax, red[i * PP + i]);
  dmax = wave_max(dmax);
  for (int i = threadIdx.x >> 6; i < m; i += blockDim.x >> 6)
    for (int j = l; j < m; j += 64)
      A[i * LD + j] = i < p && j < p ? 0.5 * (red[i * PP + j] + red[j * PP + i]) : 0.0;
  __syncthreads();
  if (chol_lds<PP, false>(p, A, 1e-13 * dmax) && threadIdx.x == 0) *flag = 1;
  inv_chol<PP>(p, A, Mb, LD);
  double* M = small + S_M * PP * PP;
  for (int i = threadIdx.x >> 6; i < PP; i += blockDim.x >> 6)
    for (int j = l; j < PP; j += 64) M[i * PP + j] = i < p && j < p ? Mb[i * LD + j] : 0.0;
}

// After a Cholesky QR pass X <- X M (M = R^{-1} in small[S_M]): C <- M^T C M, W <- M^T W.
// If the factorization was flagged as failed, M is reset to the identity instead.
template <int PP>
__global__ __launch_bounds__(WG) void k_transform_cw(double* __restrict__ small, int* __restrict__ flag) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double* T1 = PP > PP_LDS_MAX ? small + small_work_offset(PP) + 4 * PP * (PP + 1) : reinterpret_cast<double*>(lds_raw);
  double* T2 = T1 + PP * PP;
  double* M = small + S_M * PP * PP;
  double* C = small + S_C * PP * PP;
  double* W = small + S_W * PP * PP;
  if (*flag) {
    for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) M[e] = (e / PP) == (e % PP) ? 1.0 : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) *flag = 0;
    return;
  }
  wg_mm<PP>(C, false, M, false, T1);  // C M
  wg_mm<PP>(M, true, W, false, T2);   // M^T W
  __syncthreads();
  wg_mm<PP>(M, true, T1, false, C);   // M^T C M
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) W[e] = T2[e];
  __syncthreads();
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
    const int i = e / PP, j = e % PP;
    if (i < j) {
      const double v = 0.5 * (C[i * PP + j] + C[j * PP + i]);
      C[i * PP + j] = v;
      C[j * PP + i] = v;
    }
  }
}

// Rayleigh-Ritz: eig of sym(red) (p x p): eigenvalues descending into vals[0..p),
// eigenvectors as the columns of small[S_M] (stride PP, padding zero). sym(red) is indefinite:
// it is shifted by its lowest Gershgorin bound where that is negative, and the eigenvalues are the
// Rayleigh quotients of the vectors with the matrix as it came (the shifted ones less the shift
// are wrong by eps times it: small values beside large ones were lost).
template <int PP>
__global__ __launch_bounds__(dense_threads(PP)) void k_ritz(int p, const double* __restrict__ red,
                                                            double* __restrict__ small, double* __restrict__ vals) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr int LD = DLD<PP>;
  double* A = reinterpret_cast<double*>(lds_raw);
  __shared__ double lam[PP], row[PP];
  __shared__ int order[PP];
  const int m = 16 * ((p + 15) >> 4);
  diag_order(p, order, row, [&](int i) { return red[i * PP + i]; });
  for (int i = threadIdx.x >> 6; i < m; i += blockDim.x >> 6)
    for (int j = threadIdx.x & 63; j < m; j += 64)
      A[i * LD + j] =
          i < p && j < p ? 0.5 * (red[order[i] * PP + order[j]] + red[order[j] * PP + order[i]]) : 0.0;
  __syncthreads();
  for (int i = threadIdx.x; i < p; i += blockDim.x) {
    double s = -A[i * LD + i];
    for (int j = 0; j < p; ++j) s += j == i ? 0.0 : fabs(A[i * LD + j]);
    row[i] = s;
  }
  __syncthreads();
  double shift = 0.0;
  for (int i = 0; i < p; ++i) shift = fmax(shift, row[i]);
  eig_lds<PP>(p, A, order, shift);
  __syncthreads();
  const double* const B[1] = {red};
  quad_diag<PP>(m / 16, A, B, [&](int, int i, double v) { lam[i] = v; });
  __syncthreads();
  for (int i = threadIdx.x; i < p; i += blockDim.x) order[rank_desc(lam, p, i)] = i;
  __syncthreads();
  for (int i = threadIdx.x; i < p; i += blockDim.x) vals[i] = lam[order[i]];
  double* M = small + S_M * PP * PP;
  for (int i = threadIdx.x >> 6; i < PP; i += blockDim.x >> 6)
    for (int j = threadIdx.x & 63; j < PP; j += 64) M[i * PP + j] = i < p && j < p ? A[i * LD + order[j]] : 0.0;
}

// ---------------------------------------------------------------- launchers

constexpr int eig_bytes(int PP) { return eig_lds_doubles(PP) * (int)sizeof(double); }
constexpr int linesearch_bytes(int PP) { return linesearch_lds_doubles(PP) * (int)sizeof(double); }
constexpr int ritz_bytes(int PP) { return PP * (PP + 2) * (int)sizeof(double); }
constexpr int chol_bytes(int PP) { return (PP > PP_LDS_MAX ? 1 : 2) * PP * (PP + 2) * (int)sizeof(double); }

template <int PP>
static hipError_t init_pp() {
  auto lds = [](auto* f, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
  hipError_t e = lds(k_eig<PP>, eig_bytes(PP));
  if (e == hipSuccess) e = lds(k_ritz<PP>, ritz_bytes(PP));
  if (e == hipSuccess) e = lds(k_chol_inv<PP>, chol_bytes(PP));
  if (e == hipSuccess) e = lds(k_linesearch<PP>, linesearch_bytes(PP));
  if (PP > PP_LDS_MAX) return e;  // k_transform_cw uses the work area there
  if (e == hipSuccess) e = lds(k_transform_cw<PP>, 2 * PP * PP * 8);
  return e;
}

hipError_t Small::init() {
  hipError_t e = init_pp<16>();
  if (e == hipSuccess) e = init_pp<32>();
  if (e == hipSuccess) e = init_pp<64>();
  if (e == hipSuccess) e = init_pp<128>();
  return e;
}
void Small::after_grad(hipStream_t st, int PP, double* red, double* small, Scalars* sc, double* hist, int cond,
                       Partials fold) {
  hipLaunchKernelGGL(k_after_grad, dim3(1), dim3(WG), 0, st, PP, red, small, sc, hist, cond, fold);
}
void Small::after_dir(hipStream_t st, int PP, double* red, double* small, Scalars* sc, Partials fold) {
  hipLaunchKernelGGL(k_after_dir, dim3(1), dim3(WG), 0, st, PP, red, small, sc, fold);
}
void Small::eig(hipStream_t st, int PP, double* small, Scalars* sc) {
  switch (PP) {
    case 16: k_eig<16><<<1, dense_threads(16), eig_bytes(16), st>>>(small, sc); break;
    case 32: k_eig<32><<<1, dense_threads(32), eig_bytes(32), st>>>(small, sc); break;
    case 64: k_eig<64><<<1, dense_threads(64), eig_bytes(64), st>>>(small, sc); break;
    case 128: k_eig<128><<<1, dense_threads(128), eig_bytes(128), st>>>(small, sc); break;
  }
}
void Small::linesearch(hipStream_t st, int PP, double* red, double* small, Scalars* sc, double* hist,
                       int recompute_ax, bool want_mc, Partials fold) {
  const int mc = want_mc ? 1 : 0;
  auto go = [&](auto P) {
    constexpr int pp = decltype(P)::value;
    k_linesearch<pp><<<1, dense_threads(pp), linesearch_bytes(pp), st>>>(red, small, sc, hist, recompute_ax, mc, fold);
  };
  switch (PP) {
    case 16: go(std::integral_constant<int, 16>()); break;
    case 32: go(std::integral_constant<int, 32>()); break;
    case 64: go(std::integral_constant<int, 64>()); break;
    case 128: go(std::integral_constant<int, 128>()); break;
  }
}
void Small::after_update_grams(hipStream_t st, int PP, const double* red, double* small, Scalars* sc) {
  hipLaunchKernelGGL(k_after_update_grams, dim3(1), dim3(WG), 0, st, PP, red, small, sc);
}
void Small::after_refresh(hipStream_t st, int PP, const double* red, double* small, Scalars* sc, bool hold) {
  hipLaunchKernelGGL(k_after_refresh, dim3(1), dim3(WG), 0, st, PP, red, small, sc, hold ? 1 : 0);
}
void Small::chol_inv(hipStream_t st, int PP, int p, const double* red, double* small, int* flag) {
  switch (PP) {
    case 16: k_chol_inv<16><<<1, dense_threads(16), chol_bytes(16), st>>>(p, red, small, flag); break;
    case 32: k_chol_inv<32><<<1, dense_threads(32), chol_bytes(32), st>>>(p, red, small, flag); break;
    case 64: k_chol_inv<64><<<1, dense_threads(64), chol_bytes(64), st>>>(p, red, small, flag); break;
    case 128: k_chol_inv<128><<<1, dense_threads(128), chol_bytes(128), st>>>(p, red, small, flag); break;
  }
}
void Small::transform_cw(hipStream_t st, int PP, double* small, int* flag) {
  switch (PP) {
    case 16: k_transform_cw<16><<<1, WG, 2 * 16 * 16 * 8, st>>>(small, flag); break;
    case 32: k_transform_cw<32><<<1, WG, 2 * 32 * 32 * 8, st>>>(small, flag); break;
    case 64: k_transform_cw<64><<<1, WG, 2 * 64 * 64 * 8, st>>>(small, flag); break;
    case 128: k_transform_cw<128><<<1, WG, 0, st>>>(small, flag); break;
  }
}
void Small::ritz(hipStream_t st, int PP, int p, const double* red, double* small, double* out_vals) {
  switch (PP) {
    case 16: k_ritz<16><<<1, dense_threads(16), ritz_bytes(16), st>>>(p, red, small, out_vals); break;
    case 32: k_ritz<32><<<1, dense_threads(32), ritz_bytes(32), st>>>(p, red, small, out_vals); break;
    case 64: k_ritz<64><<<1, dense_threads(64), ritz_bytes(64), st>>>(p, red, small, out_vals); break;
    case 128: k_ritz<128><<<1, dense_threads(128), ritz_bytes(128), st>>>(p, red, small, out_vals); break;
  }
}

}  // namespace gsi
