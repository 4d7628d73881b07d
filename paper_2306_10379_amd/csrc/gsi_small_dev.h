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

// ---------------------------------------------------------------- line search (wave 0)

struct Terms {
  double a[TMAXP], b[TMAXP], g[TMAXP], z[TMAXP];
};

// Term of phi'(mu) = - sum over active terms of (z + d mu - b z mu^2) / (1 + b mu^2)^2,
// d = g - a b (Sec. 5.2, eq. deriv_P).
__device__ __forceinline__ double dphi_term(double a, double b, double g, double z, double mu) {
  const double d = g - a * b, den = 1.0 + b * mu * mu;
  const double r = div_nr(1.0, den);  // den >= 1
  return den < 1e300 ? (z + d * mu - b * z * mu * mu) * r * r : 0.0;
}

// Get_Mu (Algorithm 3, Sec. 5.2, Sec. 6.1): returns mu > 0 or -1 when no usable bracket.
// Called by wave 0 only; p terms (padding terms have b = 0), preal the block size for the
// activity threshold; *evals counts phi' evaluations, *bm gets the largest b.
__device__ inline double get_mu(Terms& T, int p, int preal, int* evals, double* bm) {
  // lane l holds terms l and l + 64 (the second only for p > 64)
  const int l = threadIdx.x & 63, l2 = l + 64;
  const bool two = p > 64;
  const double al = l < p ? T.a[l] : 0.0, bl = l < p ? T.b[l] : 0.0;
  const double gl = l < p ? T.g[l] : 0.0, zl = l < p ? T.z[l] : 0.0;
  const double al2 = l2 < p ? T.a[l2] : 0.0, bl2 = l2 < p ? T.b[l2] : 0.0;
  const double gl2 = l2 < p ? T.g[l2] : 0.0, zl2 = l2 < p ? T.z[l2] : 0.0;
  const double bmax = wave_max(l2 < p ? fmax(bl, bl2) : bl);
  *bm = bmax;
  int ev = 0;
  if (!(bmax > 0.0)) { *evals = 0; return -1.0; }
  const bool act = l < p && bl > preal * EPS * bmax;
  const bool act2 = l2 < p && bl2 > preal * EPS * bmax;
  // inactive terms become zero ones, so that the sums below need no test (b stays, for M)
  if (l < p && !act) T.a[l] = T.g[l] = T.z[l] = 0.0;
  if (l2 < p && !act2) T.a[l2] = T.g[l2] = T.z[l2] = 0.0;
  wave_sync();
  const bool conv = act && zl > 0.0;
  const bool conv2 = act2 && zl2 > 0.0;
  auto dphi = [&](double mu) {
    double v = act ? dphi_term(al, bl, gl, zl, mu) : 0.0;
    if (two && act2) v += dphi_term(al2, bl2, gl2, zl2, mu);
    return -wave_sum_all(v);
  };
  if (__ballot(conv || conv2) == 0) { *evals = 0; return -1.0; }
  // f(0) = -sum of active zeta
  const double f0 = dphi(0.0);
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
#pragma unroll 8
    for (int i = 0; i < p; ++i) {
      acc += dphi_term(T.a[i], T.b[i], T.g[i], T.z[i], x);
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
    fhi = dphi(hi);
    ++ev;
    while (fhi < 0.0 && widen < 60) {
      lo = hi;
      hi *= 2.0;
      fhi = dphi(hi);
      ++ev;
      ++widen;
    }
    if (fhi < 0.0) { *evals = ev; return -1.0; }
  } else {
    fhi = dphi(hi);
    ++ev;
  }
  if (fhi == 0.0) { *evals = ev; return hi; }
  double flo = dphi(lo);
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
      const double s = div_nr(fb, fa);
      if (a == c) {
        pp = 2.0 * xm * s;
        q = 1.0 - s;
      } else {
        q = div_nr(fa, fc);
        r = div_nr(fb, fc);
        pp = s * (2.0 * xm * q * (q - r) - (b - a) * (r - 1.0));
        q = (q - 1.0) * (r - 1.0) * (s - 1.0);
      }
      if (pp > 0.0) q = -q; else pp = -pp;
      if (2.0 * pp < fmin(3.0 * xm * q - fabs(tol1 * q), fabs(e * q))) {
        e = d;
        d = div_nr(pp, q);
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
    fb = dphi(b);
    ++ev;
  }
  *evals = ev;
  return b;
}


// ---------------------------------------------------------------- eigendecomposition of P^T P

// P^T P = V diag(b) V^T (Sec. 5.2) for S = small[S_S]: writes V (small[S_V]; the line search
// forms b); returns the sweep count. Warm start (warm = true): the previous V, made
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
  auto to = [](double* dst) { return [dst](int i, int j, double v) { dst[i * LD + j] = v; }; };
  auto to_sym = [](double* dst) { return [dst](int i, int j, double v) { dst[i * LD + j] = dst[j * LD + i] = v; }; };
  if (warm) {
    constexpr int LV = wide ? PP : LD;
    const double* V0 = wide ? Vg : T;
    if constexpr (!wide) {
      fill_dense(m, T, LD, [&](int i, int j) { return Vg[i * PP + j]; });
      __syncthreads();
    }
    mm_dense<PP / 16, LV, true, LV, false, true>(nb, V0, V0, [&](int i, int j, double v) {  // (3 I - V^T V) / 2
      A[i * LD + j] = A[j * LD + i] = 0.5 * ((i == j ? 3.0 : 0.0) - v);
    });
    __syncthreads();
    mm_dense<PP / 16, LV, false, LD, false>(nb, V0, A, to(V1));
    __syncthreads();
    if constexpr (wide) {
      mm_dense<PP / 16, PP, true, LD, false>(nb, S, V1, to(T));  // S is symmetric
      __syncthreads();
      mm_dense<PP / 16, LD, true, LD, false, true>(nb, V1, T, to_sym(A));
      __syncthreads();
      diag_order(p, ord, key, [&](int i) { return A[i * LD + i]; });
      fill_dense(m, T, LD, [&](int i, int j) { return A[ord[i] * LD + ord[j]]; });
      __syncthreads();
      fill_dense(m, A, LD, [&](int i, int j) { return T[i * LD + j]; });
    } else {
      fill_dense(m, T, LD, [&](int i, int j) { return S[i * PP + j]; });
      __syncthreads();
      mm_dense<PP / 16, LD, false, LD, false>(nb, T, V1, to(A));
      __syncthreads();
      mm_dense<PP / 16, LD, true, LD, false, true>(nb, V1, A, to_sym(T));
      __syncthreads();
      diag_order(p, ord, key, [&](int i) { return T[i * LD + i]; });
      fill_dense(m, A, LD, [&](int i, int j) { return T[ord[i] * LD + ord[j]]; });
    }
  } else {
    diag_order(p, ord, key, [&](int i) { return S[i * PP + i]; });
    fill_dense(m, A, LD, [&](int i, int j) { return S[ord[i] * PP + ord[j]]; });
  }
  __syncthreads();
  const int sweeps = eig_lds<PP>(p, A, ord, 0.0);
  __syncthreads();
  if (warm)
    mm_dense<PP / 16, LD, false, LD, false>(nb, V1, A, [&](int i, int j, double v) { Vg[i * PP + j] = v; });
  else
    fill_dense(m, Vg, PP, [&](int i, int j) { return A[i * LD + j]; });
  __syncthreads();
  return sweeps;
}

// ---------------------------------------------------------------- line search and retraction factor

// v_i^T B_q v_i for the leading 16 nb columns v_i of V (LDS, stride DLD<PP>) and the matrices B_q
// (global, stride PP), put(q, i, value): the line-search diagonals, Rayleigh quotients. A wave
// takes 16 columns, whose operand stays in registers for all matrices; a matrix is read by rows
// as the transposed left operand (coalesced; v^T B v = v^T B^T v) and the product's blocks go into
// the dot products from the matrix unit's registers.
template <int PP, int NQ, typename F>
__device__ __forceinline__ void quad_diag(int nb, const double* V, const double* const (&B)[NQ], F put) {
  constexpr int LD = DLD<PP>, NB = PP / 16;
  const int nw = blockDim.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  for (int jb = threadIdx.x >> 6; jb < nb; jb += nw) {
    double v[NB][4];
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int s = 0; s < 4; ++s) v[k][s] = k < nb ? V[(16 * k + 4 * s + g) * LD + 16 * jb + c] : 0.0;
    // the blocks (matrix, ib) one after the other, the next one's rows loaded before this one's
    // products
    double x[NB][4], y[NB][4];
    auto load = [&](const double* M, int ib, double (&to)[NB][4]) {
#pragma unroll
      for (int k = 0; k < NB; ++k)
        if (k < nb)
#pragma unroll
          for (int s = 0; s < 4; ++s) to[k][s] = M[(16 * k + 4 * s + g) * PP + 16 * ib + c];
    };
    if constexpr (NB <= 4) load(B[0], 0, x);
    double sum[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      double acc = 0.0;
      for (int ib = 0; ib < nb; ++ib) {
        if constexpr (NB > 4) {
          load(B[q], ib, x);  // two waves per SIMD cover each other's loads
        } else {
          if (ib + 1 < nb) load(B[q], ib + 1, y);
          else if (q + 1 < NQ) load(B[q + 1 < NQ ? q + 1 : q], 0, y);
        }
        d4 t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NB; ++k)
          if (k < nb)
#pragma unroll
            for (int s = 0; s < 4; ++s) t = mfma(x[k][s], v[k][s], t);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = fma(t[r], V[(16 * ib + g + 4 * r) * LD + 16 * jb + c], acc);
        if constexpr (NB <= 4)
#pragma unroll
          for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) x[k][s] = y[k][s];
      }
      sum[q] = acc;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      sum[q] += __shfl_xor(sum[q], 16, 64);
      sum[q] += __shfl_xor(sum[q], 32, 64);
      if (g == 0) put(q, 16 * jb + c, sum[q]);
    }
  }
}

// Exact line search (Sec. 5.2, Algorithm 3, Sec. 6.1) from V (eig_dev), C = small[S_C],
// S = small[S_S] and the Grams P^T A P (PZr) and P^T A X (PYr). On success (*sok = 1) it
// writes mu (*smu), M = small[S_M], the next C and W (small[S_C], small[S_W]) and the largest
// b (*sbmax), and with want_mc also M C_next = small[S_MC] (the right factor of the next
// gradient, G = (X - mu P) M C_next - (Y - mu Z) M, for the fused retraction pass). lds:
// linesearch_lds_doubles(PP); terms, smu, sok, sevals, sbmax in shared memory. Whole workgroup
// of dense_threads(PP).
//
// Four quadratic diagonals, Get_Mu (5 us at p = 8, 7 us at p = 64) and eight p x p products, one
// after the other, bound it. Matrices sit in LDS at the stride that keeps the operand loads free of bank conflicts
// (with a stride of PP each load hit one bank 16 times), the Grams are read coalesced, blocks
// below the diagonal of symmetric products and past p are left out: k_linesearch 108 -> 68 us at
// p = 64 (3 of them for b, the fourth diagonal), 30 -> 29 us at p = 32, 15.5 -> 15 us at p = 8, 1010
// -> 287 us at p = 128. Above PP = 64 one matrix fits LDS (V, then M in its two stages) and the
// others sit in the work area of the small buffer, always read by rows.
constexpr int linesearch_lds_doubles(int PP) { return (PP > PP_LDS_MAX ? 1 : 4) * PP * (PP + 2); }

template <int PP>
__device__ inline void linesearch_dev(const double* PZr, const double* PYr, double* small, int p, double* lds,
                                      Terms& terms, double* smu, int* sok, int* sevals, double* sbmax,
                                      bool want_mc = false) {
  constexpr int LD = DLD<PP>;
  constexpr bool wide = PP > PP_LDS_MAX;
  const int nb = (p + 15) >> 4, m = 16 * nb;
  double* work = wide ? small + small_work_offset(PP) + 4 * PP * (PP + 1) : lds;
  double *b0 = work, *b1 = work + PP * LD, *b2 = work + 2 * PP * LD;
  double* U = wide ? lds : b0;
  const double* S = small + S_S * PP * PP;
  double* C = small + S_C * PP * PP;
  double* M = small + S_M * PP * PP;
  double* W = small + S_W * PP * PP;
  double* MC = small + S_MC * PP * PP;
  const double* Vg = small + S_V * PP * PP;
  // a matrix that the following products read from LDS
  auto settle = [&](double* src) {
    if constexpr (!wide) return src;
    __syncthreads();
    fill_dense(m, lds, LD, [&](int i, int j) { return src[i * LD + j]; });
    return lds;
  };
  fill_dense(m, U, LD, [&](int i, int j) { return Vg[i * PP + j]; });
  const double* Sm = S;  // P^T P as the products read it: S^T = S
  constexpr int LDS_S = wide ? PP : LD;
  if constexpr (!wide) {
    double* b3 = work + 3 * PP * LD;
    fill_dense(m, b3, LD, [&](int i, int j) { return S[i * PP + j]; });
    Sm = b3;
  }
  for (int i = m + threadIdx.x; i < TMAXP; i += blockDim.x) terms.a[i] = terms.b[i] = terms.g[i] = terms.z[i] = 0.0;
  __syncthreads();
  // line-search diagonals (Sec. 5.2, eq. CG_linesearch_D) in the basis V; the diagonal of
  // V^T B V only needs the symmetric part of B, so the raw Grams are used. b too is a Rayleigh
  // quotient: M below needs a small b to its own last bits, also beside one 1e16 times as large
  // (a step of mu^2 b = 1e10 in one direction left X orthonormal to 1e-7 with a b to eps of the
  // largest, to 1e-3 at 1e12)
  {
    const double* const B[4] = {C, PZr, PYr, S};
    double* const to[4] = {terms.a, terms.g, terms.z, terms.b};
    quad_diag<PP>(nb, U, B, [&](int q, int i, double v) { to[q][i] = q == 2 ? -v : (q == 3 ? fmax(v, 0.0) : v); });
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    int evals = 0;
    double bmax = 0.0;
    const double mu = get_mu(terms, PP, p, &evals, &bmax);
    if (threadIdx.x == 0) {
      *smu = mu;
      *sok = mu > 0.0 && isfinite(mu);
      *sevals = evals;
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
  // (terms.a is free after Get_Mu: it holds the column factors (1 + mu^2 b)^{-1/4})
  for (int i = threadIdx.x; i < PP; i += blockDim.x) terms.a[i] = sqrt(1.0 / sqrt(1.0 + mu * mu * terms.b[i]));
  __syncthreads();
  fill_dense(m, U, LD, [&](int i, int j) { return U[i * LD + j] * terms.a[j]; });
  __syncthreads();
  mm_dense<PP / 16, LD, false, LD, true, true>(nb, U, U, [&](int i, int j, double v) { b1[i * LD + j] = b1[j * LD + i] = v; });
  const double* M0 = settle(b1);
  __syncthreads();
  mm_dense<PP / 16, LDS_S, true, LD, false>(nb, Sm, M0, [&](int i, int j, double v) {  // B M
    b2[i * LD + j] = fma(mu * mu, v, M0[i * LD + j]);
  });
  __syncthreads();
  mm_dense<PP / 16, LD, false, LD, false, true>(nb, M0, b2, [&](int i, int j, double v) {  // 3 I - M B M
    b0[i * LD + j] = b0[j * LD + i] = (i == j ? 3.0 : 0.0) - v;
  });
  __syncthreads();
  mm_dense<PP / 16, LD, false, LD, false, true>(nb, M0, b0, [&](int i, int j, double v) {
    const double h = 0.5 * v;
    b2[i * LD + j] = b2[j * LD + i] = h;
    M[i * PP + j] = M[j * PP + i] = h;
  });
  const double* Mf = settle(b2);
  __syncthreads();
  // next C = M (C - mu (P^T Y + Y^T P) + mu^2 P^T Z) M and next W = X_new^T P = -mu M S
  // (X^T P = 0 for the tangent direction; A X recursion of Sec. 6.1, eq. save_matvec)
  // (half of it by rows, so that the Grams are read coalesced, then the sum with its transpose)
  fill_dense(m, b1, LD, [&](int i, int j) {
    return 0.5 * C[i * PP + j] - mu * PYr[i * PP + j] + 0.5 * mu * mu * PZr[i * PP + j];
  });
  __syncthreads();
  fill_dense(m, b0, LD, [&](int i, int j) { return b1[i * LD + j] + b1[j * LD + i]; });
  __syncthreads();
  mm_dense<PP / 16, LD, true, LD, false>(nb, b0, Mf, [&](int i, int j, double v) { b1[i * LD + j] = v; });
  mm_dense<PP / 16, LD, false, LDS_S, false>(nb, Mf, Sm, [&](int i, int j, double v) { W[i * PP + j] = -mu * v; });
  __syncthreads();
  mm_dense<PP / 16, LD, false, LD, false, true>(nb, Mf, b1, [&](int i, int j, double v) {
    C[i * PP + j] = C[j * PP + i] = v;
    b0[i * LD + j] = b0[j * LD + i] = v;
  });
  __syncthreads();
  if (want_mc) {
    mm_dense<PP / 16, LD, false, LD, false>(nb, Mf, b0, [&](int i, int j, double v) { MC[i * PP + j] = v; });
    __syncthreads();
  }
}

}  // namespace gsi
