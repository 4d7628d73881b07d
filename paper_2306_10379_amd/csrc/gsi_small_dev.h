// Single-workgroup float64 building blocks for the p x p projected problem, shared by the
// per-iteration kernels (gsi_small.hip) and the batched persistent solver (gsi_batched.hip):
// f64 MFMA products of PP x PP matrices, the eigendecomposition of P^T P, and Get_Mu with
// Brent's method on phi'.
#pragma once
#include <math.h>

#include "gsi_dense_dev.h"
#include "gsi_device.h"
#include "gsi_state.h"

namespace gsi {

constexpr int MAXP = 64;    // block width of the batched solve and of the one-wave routines below
constexpr int TMAXP = 128;  // block width of the single-problem float64 path (two terms per lane)

// Order LDS traffic among the lanes of one wavefront (used where only wave 0 runs).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- dense PP x PP products

// Cout = alpha * op(A) op(B) for PP x PP row-major operands (any memory space), f64 MFMA,
// 16 x 16 output blocks dealt to the 4 waves. No barrier inside. The operands of a block
// are all loaded before its products: from global memory the block then waits for one
// round of loads instead of one per group of K steps (these single-workgroup kernels have
// no other waves to hide the latency).
template <int PP>
__device__ inline void wg_mm(const double* A, bool ta, const double* B, bool tb, double* Cout, double alpha = 1.0) {
  constexpr int NBK = PP / 16;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  for (int blk = w; blk < NBK * NBK; blk += 4) {
    const int ib = blk / NBK, jb = blk % NBK;
    double a[PP / 4], b[PP / 4];
#pragma unroll
    for (int s = 0; s < PP / 4; ++s) {
      const int k = 4 * s + g;
      a[s] = ta ? A[k * PP + 16 * ib + c] : A[(16 * ib + c) * PP + k];
      b[s] = tb ? B[(16 * jb + c) * PP + k] : B[k * PP + 16 * jb + c];
    }
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < PP / 4; ++s) acc = mfma(a[s], b[s], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) Cout[(16 * ib + g + 4 * r) * PP + 16 * jb + c] = alpha * acc[r];
  }
}

// out[i] = sign * sum_k V[k][i] T[k][i]  (the diagonal of V^T T), i < PP.
template <int PP>
__device__ inline void col_dots(const double* V, const double* T, double* out, double sign) {
  for (int i = threadIdx.x; i < PP; i += blockDim.x) {
    double s = 0.0;
    for (int k = 0; k < PP; ++k) s += V[k * PP + i] * T[k * PP + i];
    out[i] = sign * s;
  }
}

// ---------------------------------------------------------------- line search (wave 0)

struct Terms {
  double a[TMAXP], b[TMAXP], g[TMAXP], z[TMAXP];
  int act[TMAXP];
};

// phi'(mu) = - sum over active terms of (z + d mu - b z mu^2) / (1 + b mu^2)^2 (Sec. 5.2,
// eq. deriv_P), evaluated by wave 0 (lane i holds terms i and i + 64).
__device__ inline double dphi_term(const Terms& T, int i, double mu) {
  const double b = T.b[i], z = T.z[i], d = T.g[i] - T.a[i] * b;
  const double den = 1.0 + b * mu * mu;
  return (z + d * mu - b * z * mu * mu) / (den * den);
}
__device__ inline double dphi(const Terms& T, int p, double mu) {
  const int l = threadIdx.x & 63;
  double v = 0.0;
  if (l < p && T.act[l]) v = dphi_term(T, l, mu);
  if (l + 64 < p && T.act[l + 64]) v += dphi_term(T, l + 64, mu);
  return -wave_sum(v);
}

// Get_Mu (Algorithm 3, Sec. 5.2, Sec. 6.1): returns mu > 0 or -1 when no usable bracket.
// Called by wave 0 only; p terms (padding terms have b = 0), preal the block size for the
// activity threshold; *evals counts phi' evaluations.
__device__ inline double get_mu(Terms& T, int p, int preal, int* evals) {
  // lane l holds terms l and l + 64 (the second only for p > 64)
  const int l = threadIdx.x & 63, l2 = l + 64;
  const double bl = l < p ? T.b[l] : 0.0;
  const double bl2 = l2 < p ? T.b[l2] : 0.0;
  const double bmax = wave_max(l2 < p ? fmax(bl, bl2) : bl);
  int ev = 0;
  if (!(bmax > 0.0)) { *evals = 0; return -1.0; }
  const bool act = l < p && bl > preal * EPS * bmax;
  const bool act2 = l2 < p && bl2 > preal * EPS * bmax;
  if (l < p) T.act[l] = act ? 1 : 0;
  if (l2 < p) T.act[l2] = act2 ? 1 : 0;
  wave_sync();
  const bool conv = act && T.z[l] > 0.0;
  const bool conv2 = act2 && T.z[l2] > 0.0;
  if (__ballot(conv || conv2) == 0) { *evals = 0; return -1.0; }
  // f(0) = -sum of active zeta
  const double f0 = dphi(T, p, 0.0);
  ++ev;
  if (!(f0 < 0.0)) { *evals = ev; return -1.0; }
  // branch roots of the convex branches, without cancellation (Sec. 6.1, eqs. derv1/derv2)
  auto root = [&](int i) {
    const double b = T.b[i], z = T.z[i], d = T.g[i] - T.a[i] * b;
    const double s = sqrt(d * d + 4.0 * b * z * z);
    return d < 0.0 ? 2.0 * z / (fabs(d) + s) : (d + s) / (2.0 * b * z);
  };
  // phi' at a candidate root: the sum over every active term
  auto dphi_all = [&](double x) {
    double acc = 0.0;
    for (int i = 0; i < p; ++i) {
      if (!T.act[i]) continue;
      const double b = T.b[i], z = T.z[i], d = T.g[i] - T.a[i] * b;
      const double den = 1.0 + b * x * x;
      acc += (z + d * x - b * z * x * x) / (den * den);
    }
    return -acc;
  };
  // every lane evaluates its own candidates
  const double xi = conv ? root(l) : INFINITY;
  const double xi2 = conv2 ? root(l2) : INFINITY;
  const double fxi = conv ? dphi_all(xi) : -1.0;
  const double fxi2 = conv2 ? dphi_all(xi2) : -1.0;
  ev += 1;
  // hi: smallest root with phi' >= 0; lo: largest root below hi (or 0)
  double hi = (conv && fxi >= 0.0) ? xi : INFINITY;
  if (conv2 && fxi2 >= 0.0) hi = fmin(hi, xi2);
  for (int o = 32; o > 0; o >>= 1) hi = fmin(hi, __shfl_xor(hi, o, 64));
  double lo = (conv && xi < hi) ? xi : 0.0;
  if (conv2 && xi2 < hi) lo = fmax(lo, xi2);
  for (int o = 32; o > 0; o >>= 1) lo = fmax(lo, __shfl_xor(lo, o, 64));
  double fhi;
  if (hi == INFINITY) {
    int widen = 0;
    hi = 2.0 * (lo > 0.0 ? lo : 1.0);
    fhi = dphi(T, p, hi);
    ++ev;
    while (fhi < 0.0 && widen < 60) {
      lo = hi;
      hi *= 2.0;
      fhi = dphi(T, p, hi);
      ++ev;
      ++widen;
    }
    if (fhi < 0.0) { *evals = ev; return -1.0; }
  } else {
    fhi = dphi(T, p, hi);
    ++ev;
  }
  if (fhi == 0.0) { *evals = ev; return hi; }
  double flo = dphi(T, p, lo);
  ++ev;
  if (flo == 0.0) { *evals = ev; return lo; }
  // Brent's method (Brent 1973, ch. 4): inverse quadratic interpolation / secant steps
  // safeguarded by bisection, on phi' over [lo, hi] with flo < 0 < fhi.
  double a = lo, b = hi, c = lo, fa = flo, fb = fhi, fc = flo;
  double d = b - a, e = d;
  for (int it = 0; it < 200; ++it) {
    if ((fb > 0.0 && fc > 0.0) || (fb < 0.0 && fc < 0.0)) {
      c = a; fc = fa; d = b - a; e = d;
    }
    if (fabs(fc) < fabs(fb)) {
      a = b; b = c; c = a;
      fa = fb; fb = fc; fc = fa;
    }
    const double tol1 = 2.0 * EPS * fabs(b) + 1e-300;
    const double xm = 0.5 * (c - b);
    if (fabs(xm) <= tol1 || fb == 0.0) break;
    if (fabs(e) >= tol1 && fabs(fa) > fabs(fb)) {
      double pp, q, r;
      const double s = fb / fa;
      if (a == c) {
        pp = 2.0 * xm * s;
        q = 1.0 - s;
      } else {
        q = fa / fc;
        r = fb / fc;
        pp = s * (2.0 * xm * q * (q - r) - (b - a) * (r - 1.0));
        q = (q - 1.0) * (r - 1.0) * (s - 1.0);
      }
      if (pp > 0.0) q = -q; else pp = -pp;
      if (2.0 * pp < fmin(3.0 * xm * q - fabs(tol1 * q), fabs(e * q))) {
        e = d;
        d = pp / q;
      } else {
        d = xm;
        e = d;
      }
    } else {
      d = xm;
      e = d;
    }
    a = b;
    fa = fb;
    b += fabs(d) > tol1 ? d : (xm > 0.0 ? tol1 : -tol1);
    fb = dphi(T, p, b);
    ++ev;
  }
  *evals = ev;
  return b;
}


// ---------------------------------------------------------------- eigendecomposition of P^T P

// P^T P = V diag(b) V^T (Sec. 5.2) for S = small[S_S]: writes V (small[S_V]) and b
// (small[S_VEC ...]); returns the sweep count. Warm start (warm = true): the previous V, made
// orthonormal again by one Newton-Schulz step V <- V (3 I - V^T V) / 2, turns S into a nearly
// diagonal V^T S V when the directions change little from step to step.
// lds: eig_lds_doubles(PP) doubles; above PP = 64 only the matrix that is decomposed fits
// there, and V and the products' temporaries sit in the work area of the small buffer. Whole
// workgroup of dense_threads(PP).
constexpr int eig_lds_doubles(int PP) { return (PP > PP_LDS_MAX ? 1 : 3) * PP * (PP + 2); }

template <int PP>
__device__ inline int eig_dev(double* small, int p, bool warm, double* lds) {
  constexpr int LD = DLD<PP>;
  constexpr bool wide = PP > PP_LDS_MAX;
  __shared__ double key[PP];
  __shared__ int ord[PP];
  const int nb = (p + 15) >> 4, m = 16 * nb;
  double* A = lds;
  double* V1 = wide ? small + small_work_offset(PP) : lds + PP * LD;
  double* T = V1 + PP * LD;
  const double* S = small + S_S * PP * PP;
  double* Vg = small + S_V * PP * PP;
  double* b = small + S_VEC * PP * PP;
  // the leading m x m block of f(i, j), 64 columns to a wave
  auto fill = [&](double* dst, int ld, auto f) {
    for (int i = threadIdx.x >> 6; i < m; i += blockDim.x >> 6)
      for (int j = threadIdx.x & 63; j < m; j += 64) dst[i * ld + j] = f(i, j);
  };
  if (warm) {
    const double* V0 = Vg;
    int ldv = PP;
    if constexpr (!wide) {
      fill(T, LD, [&](int i, int j) { return Vg[i * PP + j]; });
      V0 = T;
      ldv = LD;
      __syncthreads();
    }
    mm_lds(nb, V0, ldv, true, V0, ldv, false, A, LD);
    __syncthreads();
    fill(A, LD, [&](int i, int j) { return 0.5 * ((i == j ? 3.0 : 0.0) - A[i * LD + j]); });
    __syncthreads();
    mm_lds(nb, V0, ldv, false, A, LD, false, V1, LD);
    __syncthreads();
    if constexpr (wide) {
      mm_lds(nb, S, PP, false, V1, LD, false, T, LD);
      __syncthreads();
      mm_lds(nb, V1, LD, true, T, LD, false, A, LD);
    } else {
      fill(T, LD, [&](int i, int j) { return S[i * PP + j]; });
      __syncthreads();
      mm_lds(nb, T, LD, false, V1, LD, false, A, LD);
      __syncthreads();
      mm_lds(nb, V1, LD, true, A, LD, false, T, LD);
    }
    __syncthreads();
    // symmetric to the last bit, sorted by the diagonal
    if constexpr (wide) {
      diag_order(p, ord, key, [&](int i) { return A[i * LD + i]; });
      fill(T, LD, [&](int i, int j) { return 0.5 * (A[ord[i] * LD + ord[j]] + A[ord[j] * LD + ord[i]]); });
      __syncthreads();
      fill(A, LD, [&](int i, int j) { return T[i * LD + j]; });
    } else {
      diag_order(p, ord, key, [&](int i) { return T[i * LD + i]; });
      fill(A, LD, [&](int i, int j) { return 0.5 * (T[ord[i] * LD + ord[j]] + T[ord[j] * LD + ord[i]]); });
    }
  } else {
    diag_order(p, ord, key, [&](int i) { return S[i * PP + i]; });
    fill(A, LD, [&](int i, int j) { return S[ord[i] * PP + ord[j]]; });
  }
  __syncthreads();
  const int sweeps = eig_lds<PP>(p, A, ord, 0.0, b);
  __syncthreads();
  if (warm)
    mm_lds(nb, V1, LD, false, A, LD, false, Vg, PP);
  else
    fill(Vg, PP, [&](int i, int j) { return A[i * LD + j]; });
  for (int i = threadIdx.x; i < PP; i += blockDim.x) b[i] = i < p ? fmax(b[i], 0.0) : 0.0;
  __syncthreads();
  return sweeps;
}

// ---------------------------------------------------------------- line search and retraction factor

// Exact line search (Sec. 5.2, Algorithm 3, Sec. 6.1) from V, b (eig_dev), C = small[S_C],
// S = small[S_S] and the Grams P^T A P (PZr) and P^T A X (PYr). On success (*sok = 1) it
// writes mu (*smu), M = small[S_M], the next C and W (small[S_C], small[S_W]) and the largest
// b (*sbmax), and with want_mc also M C_next = small[S_MC] (the right factor of the next
// gradient, G = (X - mu P) M C_next - (Y - mu Z) M, for the fused retraction pass). lds: 4 PP^2
// doubles; terms, smu, sok, sevals, sbmax in shared memory. Whole workgroup.
template <int PP>
__device__ inline void linesearch_dev(const double* PZr, const double* PYr, double* small, int p, double* lds,
                                      Terms& terms, double* smu, int* sok, int* sevals, double* sbmax,
                                      bool want_mc = false) {
  double* V = lds;
  double* Mc = V + PP * PP;
  double* T1 = Mc + PP * PP;
  double* T2 = T1 + PP * PP;
  const double* S = small + S_S * PP * PP;
  double* C = small + S_C * PP * PP;
  const double* bvec = small + S_VEC * PP * PP;
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) V[e] = small[S_V * PP * PP + e];
  for (int i = threadIdx.x; i < TMAXP; i += blockDim.x) terms.b[i] = i < PP ? bvec[i] : 0.0;
  __syncthreads();
  // line-search diagonals (Sec. 5.2, eq. CG_linesearch_D) in the basis V; the diagonal of
  // V^T B V only needs the symmetric part of B, so the raw Grams are used
  wg_mm<PP>(C, false, V, false, T1);
  wg_mm<PP>(PZr, false, V, false, T2);
  __syncthreads();
  col_dots<PP>(V, T1, terms.a, 1.0);
  col_dots<PP>(V, T2, terms.g, 1.0);
  wg_mm<PP>(PYr, false, V, false, Mc);
  __syncthreads();
  col_dots<PP>(V, Mc, terms.z, -1.0);
  __syncthreads();
  if (threadIdx.x < 64) {
    int evals = 0;
    const double mu = get_mu(terms, PP, p, &evals);
    if (threadIdx.x == 0) {
      *smu = mu;
      *sok = mu > 0.0 && isfinite(mu);
      *sevals = evals;
      double bmax = 0.0;
      for (int i = 0; i < p; ++i) bmax = fmax(bmax, terms.b[i]);
      *sbmax = bmax;
    }
  }
  __syncthreads();
  if (!*sok) return;
  const double mu = *smu;
  // M = V diag((1 + mu^2 b)^{-1/2}) V^T (Sec. 5.2, eq. Xnew_P). V is orthogonal only to
  // about (number of rotations) * eps, which would let X(mu) drift from orthonormality
  // step after step; one Newton step for the inverse square root of B = I + mu^2 S,
  // M <- M (3 I - M B M) / 2, restores M B M = I to second order.
  // (terms.a is free after Get_Mu: it holds the PP column factors (1 + mu^2 b)^{-1/2})
  for (int i = threadIdx.x; i < PP; i += blockDim.x) terms.a[i] = 1.0 / sqrt(1.0 + mu * mu * terms.b[i]);
  __syncthreads();
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) T1[e] = V[e] * terms.a[e % PP];
  __syncthreads();
  wg_mm<PP>(T1, false, V, true, Mc);  // Mc = V D V^T
  __syncthreads();
  wg_mm<PP>(S, false, Mc, false, T1);  // T1 = S M
  __syncthreads();
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) T1[e] = Mc[e] + mu * mu * T1[e];  // B M
  __syncthreads();
  wg_mm<PP>(Mc, false, T1, false, T2);  // M B M
  __syncthreads();
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) T2[e] = ((e / PP) == (e % PP) ? 3.0 : 0.0) - T2[e];
  __syncthreads();
  wg_mm<PP>(Mc, false, T2, false, T1);  // M (3I - M B M)
  __syncthreads();
  double* M = small + S_M * PP * PP;
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
    const int i = e / PP, j = e % PP;
    const double v = 0.25 * (T1[i * PP + j] + T1[j * PP + i]);
    Mc[e] = v;
    M[e] = v;
  }
  __syncthreads();
  // next C = M (C - mu (P^T Y + Y^T P) + mu^2 P^T Z) M and next W = X_new^T P = -mu M S
  // (X^T P = 0 for the tangent direction; A X recursion of Sec. 6.1, eq. save_matvec)
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
    const int i = e / PP, j = e % PP;
    T2[e] = C[e] - mu * (PYr[e] + PYr[j * PP + i]) + 0.5 * mu * mu * (PZr[e] + PZr[j * PP + i]);
  }
  __syncthreads();
  wg_mm<PP>(Mc, false, T2, false, T1);
  __syncthreads();
  wg_mm<PP>(T1, false, Mc, false, T2);
  double* W = small + S_W * PP * PP;
  wg_mm<PP>(Mc, false, S, false, W, -mu);
  __syncthreads();
  for (int e = threadIdx.x; e < PP * PP; e += blockDim.x) {
    const int i = e / PP, j = e % PP;
    C[e] = 0.5 * (T2[e] + T2[j * PP + i]);
  }
  __syncthreads();
  if (want_mc) {
    wg_mm<PP>(Mc, false, C, false, small + S_MC * PP * PP);
    __syncthreads();
  }
}

}  // namespace gsi
