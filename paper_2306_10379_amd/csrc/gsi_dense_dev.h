// Dense symmetric p x p building blocks of one workgroup, p <= 128: products on f64 MFMA, a
// blocked Cholesky factorization and an eigensolver (one-sided Jacobi on the Cholesky factor,
// columns in registers). Matrices sit in LDS with row stride DLD<PP> = PP + 2: the 16 rows
// that one MFMA operand load touches then start 4 banks apart, and the four k-columns of the
// lane groups fill the banks between, so the loads are free of conflicts (a stride of PP puts
// all 16 rows on one bank).
#pragma once
#include <math.h>

#include <type_traits>

#include "gsi_device.h"
#include "gsi_state.h"

namespace gsi {

constexpr double EPS = 2.220446049250313e-16;

template <int PP>
constexpr int DLD = PP + 2;

// Threads of the single-workgroup p x p kernels: a wave per 16 columns of the eigensolver, at
// least the 4 waves that keep the four SIMDs' matrix cores busy.
constexpr int dense_threads(int PP) { return PP > 64 ? 512 : 256; }

// Reciprocal square root in float64: the hardware approximation (24 bits or more) refined by
// one third-order step, y (1 + e / 2 + 3 e^2 / 8) with e = 1 - x y^2, whose error e^3 is below
// the last bit; for positive normal arguments.
__device__ __forceinline__ double rsq_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// x / y by the hardware reciprocal and one third-order step (y normal; otherwise it may give
// no number).
__device__ __forceinline__ double div_nr(double x, double y) {
  const double r = __builtin_amdgcn_rcp(y), e = fma(-y, r, 1.0);
  return x * fma(r * e, 1.0 + e, r);
}

// ---------------------------------------------------------------- products

// op(A) op(B) on the leading 16 nb x 16 nb blocks (nb <= NB), row strides LDA and LDB (any
// memory space); put(i, j, v) takes each entry. SYM: the product is symmetric, only blocks on
// and above the diagonal are formed, and put sees i <= j (to store both). No barrier inside.
//
// A wave takes whole columns of 16 x 16 blocks: the right operand of 16 of k is loaded once for
// all of them, their accumulators are independent MFMA chains, and the loads of the next 16 of k
// are issued before these multiply. Strides and transposes are compile-time values, so that
// loads are one base address and immediate offsets. 7.0k clocks at p = 64, against 4.1k of MFMA
// issue on the four SIMDs (block by block: 8.2k).
template <int NB, int LDA, bool TA, int LDB, bool TB, bool SYM = false, typename F>
__device__ __forceinline__ void mm_dense(int nb, const double* A, const double* B, F put) {
  constexpr int SA = TA ? LDA : 1, SB = TB ? 1 : LDB;  // steps of k
  constexpr int IA = TA ? 16 : 16 * LDA;               // step of a block row
  const int nw = blockDim.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  for (int jb = threadIdx.x >> 6; jb < nb; jb += nw) {
    const int ni = SYM ? jb + 1 : nb;
    const double* a = A + (TA ? c : c * LDA) + g * SA;
    const double* b = B + (TB ? (16 * jb + c) * LDB : 16 * jb + c) + g * SB;
    d4 acc[NB];
    double av[NB][4], bv[4];
    auto load = [&](double (&x)[NB][4], double (&y)[4]) {
#pragma unroll
      for (int s = 0; s < 4; ++s) y[s] = b[4 * s * SB];
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (i < ni)
#pragma unroll
          for (int s = 0; s < 4; ++s) x[i][s] = a[i * IA + 4 * s * SA];
    };
    auto mul = [&]() {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (i < ni)
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[i] = mfma(av[i][s], bv[s], acc[i]);
    };
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i] = d4{0.0, 0.0, 0.0, 0.0};
    load(av, bv);
    for (int k = 1; k < nb; ++k) {
      a += 16 * SA;
      b += 16 * SB;
      if constexpr (NB > 4) {  // two waves per SIMD cover each other's loads; no room for both
        mul();
        load(av, bv);
      } else {
        double an[NB][4], bn[4];
        load(an, bn);
        mul();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          bv[s] = bn[s];
#pragma unroll
          for (int i = 0; i < NB; ++i) av[i][s] = an[i][s];
        }
      }
    }
    mul();
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i < ni)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + g + 4 * r, col = 16 * jb + c;
          if (!SYM || row <= col) put(row, col, acc[i][r]);
        }
  }
}

// dst[i ld + j] = f(i, j) on the leading m x m square, 64 columns to a wave.
template <typename F>
__device__ __forceinline__ void fill_dense(int m, double* dst, int ld, F f) {
  for (int i = threadIdx.x >> 6; i < m; i += blockDim.x >> 6)
    for (int j = threadIdx.x & 63; j < m; j += 64) dst[i * ld + j] = f(i, j);
}

// ---------------------------------------------------------------- Cholesky

__device__ __forceinline__ double readlane_d(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Lower Cholesky factor in place of the leading p x p block of A (LDS, stride DLD<PP>, both
// triangles given, rows and columns p .. 16 ceil(p/16) zero). What is left above the diagonal
// is not part of it. A pivot not above `floor` (or NaN) is replaced by it (FIX), or reported, as
// is one that is not finite: returns true in wave 0 when there was one (the factor is then of
// no use).
//
// 16 columns at a time: wave 0 factors the panel with a row per lane (two at PP = 128), the
// pivots and multipliers broadcast by v_readlane, with no barrier or LDS traffic inside the
// panel; the trailing blocks are updated by all waves on MFMA. A column-at-a-time
// factorization in LDS, with three barriers a column, took 209 us at p = 64 with its inverse.
template <int PP, bool FIX>
__device__ __forceinline__ bool chol_lds(int p, double* A, double floor) {
  constexpr int LD = DLD<PP>, NR = PP > 64 ? 2 : 1;
  const int nb = (p + 15) >> 4, nw = blockDim.x >> 6, w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int g = l >> 4, c = l & 15;
  bool bad = false;
  for (int kb = 0; kb < nb; ++kb) {
    const int c0 = 16 * kb;
    if (w == 0) {
      double a[NR][16];
#pragma unroll
      for (int h = 0; h < NR; ++h) {
        const int row = l + 64 * h;
        const bool in = row >= c0 && row < 16 * nb;
#pragma unroll
        for (int j = 0; j < 16; ++j) a[h][j] = in ? A[row * LD + c0 + j] : 0.0;
      }
      auto panel = [&](auto H) {
        constexpr int h = decltype(H)::value;  // the pivot rows are rows c0 .. c0 + 15 of half h
        const int l0 = c0 - 64 * h;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          double piv = readlane_d(a[h][j], l0 + j);
          if constexpr (FIX) {
            piv = fmax(piv, floor);
            a[h][j] = l == l0 + j ? piv : a[h][j];
          } else {
            bad |= c0 + j < p && !(piv > floor && piv < INFINITY);
          }
          // a zero matrix, and the padding columns of the last panel: zero factor
          const double rs = piv > 0.0 ? rsq_nr(piv) : 0.0;
#pragma unroll
          for (int q = 0; q < NR; ++q) a[q][j] *= rs;
#pragma unroll
          for (int k = j + 1; k < 16; ++k) {
            const double m = readlane_d(a[h][j], l0 + k);
#pragma unroll
            for (int q = 0; q < NR; ++q) a[q][k] = fma(-a[q][j], m, a[q][k]);
          }
          // column by column: the scheduler would sink the updates and keep all broadcasts
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (NR == 1 || c0 < 64)
        panel(std::integral_constant<int, 0>());
      else
        panel(std::integral_constant<int, NR - 1>());
#pragma unroll
      for (int h = 0; h < NR; ++h) {
        const int row = l + 64 * h;
        if (row >= c0 && row < 16 * nb)
#pragma unroll
          for (int j = 0; j < 16; ++j) A[row * LD + c0 + j] = a[h][j];
      }
    }
    __syncthreads();
    // trailing blocks (ib, jb), kb < jb <= ib: A -= L L^T
    const int nt = nb - 1 - kb;
    for (int t = w; t < nt * (nt + 1) / 2; t += nw) {
      int ib = 0, r = t;
      while (r > ib) r -= ++ib;
      const int i0 = 16 * (kb + 1 + ib), j0 = 16 * (kb + 1 + r);
      d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc = mfma(A[(i0 + c) * LD + c0 + 4 * s + g], A[(j0 + c) * LD + c0 + 4 * s + g], acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) A[(i0 + g + 4 * q) * LD + j0 + c] -= acc[q];
    }
    __syncthreads();
  }
  return bad;
}

// M = L^{-T} (upper triangular, all of its leading 16 ceil(p/16) square written, padding zero)
// for the factor L that chol_lds left in A; M: stride ldm, LDS or global. Whole workgroup,
// barriers inside; the caller puts one after.
//
// X = L^{-1} by block rows, M[j][i] = X[i][j]: 16 lanes invert each diagonal block, a column
// each; block row i is then -X_ii sum_k L_ik X_kj on MFMA, whose inner sum leaves the matrix
// unit in the layout that the product with X_ii takes it in.
template <int PP>
__device__ __forceinline__ void inv_chol(int p, const double* A, double* M, int ldm) {
  constexpr int LD = DLD<PP>;
  const int nb = (p + 15) >> 4, nw = blockDim.x >> 6, w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int g = l >> 4, c = l & 15;
  if (const int kb = threadIdx.x >> 4; kb < nb) {
    const int d = 16 * kb;
    double x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double s = i == c ? 1.0 : 0.0;
#pragma unroll
      for (int k = 0; k < i; ++k) s = fma(-A[(d + i) * LD + d + k], x[k], s);
      x[i] = d + i < p ? s / A[(d + i) * LD + d + i] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) M[(d + c) * ldm + d + i] = x[i];
  }
  for (int t = w; t < nb * nb; t += nw) {  // zero below the diagonal
    const int ib = t / nb, jb = t - ib * nb;
    if (ib > jb)
      for (int r = g; r < 16; r += 4) M[(16 * ib + r) * ldm + 16 * jb + c] = 0.0;
  }
  __syncthreads();
  for (int i = 1; i < nb; ++i) {
    for (int j = w; j < i; j += nw) {
      d4 t = {0.0, 0.0, 0.0, 0.0};
      for (int k = j; k < i; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          t = mfma(A[(16 * i + c) * LD + 16 * k + 4 * s + g], M[(16 * j + c) * ldm + 16 * k + 4 * s + g], t);
      d4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s) x = mfma(M[(16 * i + 4 * s + g) * ldm + 16 * i + c], t[s], x);
#pragma unroll
      for (int r = 0; r < 4; ++r) M[(16 * j + c) * ldm + 16 * i + g + 4 * r] = -x[r];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- eigensolver

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  return __hiloint2double(dpp_i<CTRL>(__double2hiint(v)), dpp_i<CTRL>(__double2loint(v)));
}
// lane l takes the value of lane l ^ M, M = 1, 2, 4, 7 (within groups of 8 lanes)
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_XOR3 = 0x1B, DPP_XOR7 = 0x141, DPP_ROR8 = 0x128;
template <typename U, int M>
__device__ __forceinline__ U lane_xor(U v) {
  auto one = [](U x, auto C) {
    if constexpr (sizeof(U) == 8) return dpp_d<decltype(C)::value>(x);
    else return dpp_i<decltype(C)::value>(x);
  };
  if constexpr (M == 1) return one(v, std::integral_constant<int, DPP_XOR1>());
  else if constexpr (M == 2) return one(v, std::integral_constant<int, DPP_XOR2>());
  else if constexpr (M == 7) return one(v, std::integral_constant<int, DPP_XOR7>());
  else return one(one(v, std::integral_constant<int, DPP_XOR7>()), std::integral_constant<int, DPP_XOR3>());
}

// Each v[k] summed over the 8 lanes that differ in lane bits 3, 4, 5; every lane gets the same
// bits. The K sums go step by step side by side (left alone, the scheduler puts the chains one
// after the other).
template <int K>
__device__ __forceinline__ void sum_rows8(double (&v)[K]) {
  double o[K];
#pragma unroll
  for (int k = 0; k < K; ++k) o[k] = dpp_d<DPP_ROR8>(v[k]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += o[k];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v[k]), __double2loint(v[k]), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v[k]), __double2hiint(v[k]), false, false);
    v[k] = __hiloint2double(hi[0], lo[0]);
    o[k] = __hiloint2double(hi[1], lo[1]);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += o[k];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v[k]), __double2loint(v[k]), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v[k]), __double2hiint(v[k]), false, false);
    v[k] = __hiloint2double(hi[0], lo[0]);
    o[k] = __hiloint2double(hi[1], lo[1]);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += o[k];
}

// Sum over the 64 lanes; every lane gets the same bits.
__device__ __forceinline__ double wave_sum_all(double v) {
  v += dpp_d<DPP_XOR1>(v);
  v += dpp_d<DPP_XOR2>(v);
  v += dpp_d<DPP_XOR7>(v);
  double o[1] = {v};
  sum_rows8(o);
  return o[0];
}

// A wave's 8 column pairs (x, y) of eig_lds: pair q = lane mod 8, R rows a lane.
template <int R>
struct ColPairs {
  double x[R], y[R];
  double a, b;      // squared norms of x and y
  int ix, iy;       // column numbers
  float cm, em;     // largest cosine rotated, largest disturbance of the other cosines
  float tol;

  __device__ __forceinline__ void norms() {
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[0] = fma(x[r], x[r], v[0]);
      v[1] = fma(y[r], y[r], v[1]);
    }
    sum_rows8(v);
    a = v[0];
    b = v[1];
  }
  // Rotates every pair whose cosine is above the threshold, by the angle theta of at most 45 degrees
  // with tan 2 theta = 2 c / d, c = x.y, d = |y|^2 - |x|^2. The angle enters as h = tan(theta / 2),
  //   s = 2 h / (1 + h^2),  x <- x - s (y + h x),  y <- y + s (x - h y)
  // (Rutishauser 1966), whose cosine is 1 - s h: rounding h changes the angle only, rounding s
  // the columns' norms by s h of it. With a rounded cosine and sine the norms grew by 2e-17 a
  // rotation, all in one direction (9e-15 of their squares at p = 64), and the vectors were off by
  // up to 6e-15 at p = 128; in this form 2e-16 and 2e-15. h is taken in float32 (short latencies; a
  // rotation then leaves 1e-7 of the cosine it meets instead of nothing, which the next sweep or
  // the stop rule accounts for; the errors against 64 bits are the same with a float64 angle).
  // The norms are updated, and formed again once per block of pairings.
  __device__ __forceinline__ void rotate() {
    double v[1] = {0.0};
#pragma unroll
    for (int r = 0; r < R; ++r) v[0] = fma(x[r], y[r], v[0]);
    const float fa = (float)a, fb = (float)b, fd = (float)(b - a);
    // zero columns: finite (fa + fb is 1e-15 or more otherwise, see eig_lds)
    const float s = __builtin_amdgcn_rcpf(fmaxf(fa + fb, 1e-30f)), g = __builtin_amdgcn_rsqf(fa * fb);
    const float vd = fabsf(fd * s), vd2 = vd * vd, big = fmaxf(fa, fb) * g, s2 = copysignf(2.f * s, fd);
    sum_rows8(v);
    const float fc = (float)v[0];
    const float u = fc * s2, co = fabsf(fc) * g;
    const bool rot = co > tol;  // false for zero columns (not a number)
    const float ri = rot ? __builtin_amdgcn_rsqf(fmaf(u, u, vd2)) : 0.f;  // 0: h and tan theta are 0
    const float k = fmaf(0.5f, vd * ri, 0.5f), rk = __builtin_amdgcn_rsqf(k);  // cos^2 theta, 1 / cos theta
    const float st = u * ri * (0.5f * rk), c1 = fmaf(k, rk, 1.f);              // sin theta, 1 + cos theta
    const float h = st * __builtin_amdgcn_rcpf(c1), t = st * rk;
    cm = fmaxf(cm, rot ? co : 0.f);
    em = fmaxf(em, fabsf(t) * big);
    // s = 2 h / (1 + h^2) from 1 / (1 + h^2) = (1 + cos theta) / 2 to float32, one third-order step
    const double hd = h, cd = c1, er = fma(fma(hd, hd, 1.0), -0.5 * cd, 1.0), m = hd * cd;
    const double sn = fma(m, fma(er, er, er), m), tc = (double)(t * fc);
    a -= tc;
    b += tc;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double xr = x[r], yr = y[r];
      x[r] = fma(-sn, fma(hd, xr, yr), xr);
      y[r] = fma(sn, fma(-hd, yr, xr), yr);
    }
  }
  // y from lane ^ M
  template <int M>
  __device__ __forceinline__ void move() {
#pragma unroll
    for (int r = 0; r < R; ++r) y[r] = lane_xor<double, M>(y[r]);
    b = lane_xor<double, M>(b);
    iy = lane_xor<int, M>(iy);
  }
  // x of the lanes with bit M set trades places with y of the others: the columns of x, and
  // those of y, then face each other
  template <int M>
  __device__ __forceinline__ void split() {
    const bool hi = (threadIdx.x & M) != 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double got = lane_xor<double, M>(hi ? x[r] : y[r]);
      x[r] = hi ? got : x[r];
      y[r] = hi ? y[r] : got;
    }
    const double gotn = lane_xor<double, M>(hi ? a : b);
    a = hi ? gotn : a;
    b = hi ? b : gotn;
    const int goti = lane_xor<int, M>(hi ? ix : iy);
    ix = hi ? goti : ix;
    iy = hi ? iy : goti;
  }
  // every x with every y of its group of 8 lanes (full: also the x, and the y, among
  // themselves). Pairings 0, 1, 3, 2 (lane xor) of a group of 4 make one body.
  __device__ __forceinline__ void meet(bool full) {
    const int segs = full ? 3 : 2;
    norms();
    for (int i = 0; i < segs; ++i) {
      rotate();
      move<1>();
      rotate();
      move<2>();
      rotate();
      move<1>();
      rotate();
      if (i == 0) move<7>();
      else if (full && i == 1) split<4>();
    }
    if (!full) return;
    split<2>();
    rotate();
    move<1>();
    rotate();
    split<1>();
    rotate();
  }
};

// Position of v[i] among v[0..p) in descending order (equal values by index, NaN last).
__device__ inline int rank_desc(const double* v, int p, int i) {
  auto key = [&](int j) { return v[j] == v[j] ? v[j] : -INFINITY; };
  const double x = key(i);
  int r = 0;
  for (int j = 0; j < p; ++j) r += key(j) > x || (j < i && key(j) == x) ? 1 : 0;
  return r;
}

// The order of a matrix's diagonal d(i), i < p, from the largest down, for eig_lds: the
// factor of a matrix sorted that way has its large columns first and nearly orthogonal columns
// when the matrix is graded (8 against 5 sweeps on a Gram matrix graded over 3 decades, and 14
// when it is sorted the other way). ord and key: LDS, 16 ceil(p/16) entries. Ends with a barrier.
template <typename F>
__device__ __forceinline__ void diag_order(int p, int* ord, double* key, F d) {
  for (int i = threadIdx.x; i < 16 * ((p + 15) >> 4); i += blockDim.x) {
    if (i < p) key[i] = d(i);
    else ord[i] = i;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < p; i += blockDim.x) ord[rank_desc(key, p, i)] = i;
  __syncthreads();
}

// Eigendecomposition B = U diag(lam) U^T of a symmetric p x p matrix. A (LDS, stride DLD<PP>,
// both triangles, rows and columns p .. 16 ceil(p/16) zero) holds B with its rows and columns
// in the order ord (LDS, from diag_order): A[i][j] = B[ord[i]][ord[j]]. It is replaced by U,
// column j the eigenvector that the rotations grew out of column ord[j] of B (columns p .. are
// unit vectors); the eigenvalues are its Rayleigh quotients with B (quad_diag). B + shift I must
// be positive semidefinite up to rounding: shift = 0 for a Gram matrix. Returns the number of
// sweeps. Whole workgroup, dense_threads(PP) threads; the caller puts a barrier before and after.
//
// A + (shift + delta) I = L L^T (delta a few ulps of the largest diagonal entry, the floor of
// the pivots too, so that a rank-deficient Gram has a factor), then rotations from the right
// make the columns of L orthogonal (one-sided Jacobi on the Cholesky factor, Veselic and Hari
// 1989): L J = U Sigma, so the columns' directions are the eigenvectors, with no second matrix to
// rotate and no row updates. Their squared norms are the eigenvalues plus shift + delta, to eps of
// the largest: they keep nothing of an eigenvalue below that.
//
// What bounds it is latency: a chain of ~p rounds per sweep, each the three dot products of a
// column pair, one rotation and its application. Wave w holds 16 columns in registers, pair q
// of lanes q + 8 g (lane group g holds the rows r = g mod 8), so the dot products are sums in
// registers and three cross-lane adds, and the column pairs of a wave meet by DPP moves of one
// column (lane xor 1, 2, 7 walk through all 8 pairings): no LDS and no barrier. The blocks of 8
// columns go round the waves (circle tournament) through LDS once every 8 rounds. The
// two-sided Jacobi with the matrix and V in LDS that this replaces moved both every round:
// k_eig 526 -> 171 us at p = 64 (35 x 40 x 25 Laplacian, 25 iterations from a random block),
// 113 -> 63 us at p = 32, 28 -> 26 us at p = 8, 22 -> 1.2 ms at p = 128 (where half the
// matrix's traffic went to memory). A round takes 510 clocks at p <= 16 and 760 at p = 64, a
// sweep p - 1 of them (some 10 of it for the half angle, against a cosine and sine).
//
// A pair is rotated when |x.y| > eps |x| |y|. A larger bound saves nothing, since every pairing is
// computed whether it rotates or not; with sqrt(PP) eps the vectors were orthogonal to 1.8e-15 at p =
// 64 and 2.7e-15 at p = 128 instead of 5e-16. The sweeps stop after one in which the
// largest cosine met times the largest disturbance of a rotation on the other cosines
// (|tan| times the ratio of the columns' norms) is below eps: what that sweep leaves is then
// below the threshold, and no confirming sweep is run.
template <int PP>
__device__ __forceinline__ int eig_lds(int p, double* A, const int* ord, double shift) {
  constexpr int LD = DLD<PP>, R = PP / 8, NW = PP / 16;
  __shared__ int ids[2 * NW][8];
  __shared__ float stat[NW][2];
  const int nw = (p + 15) >> 4, w = threadIdx.x >> 6, l = threadIdx.x & 63, q = l & 7, g = l >> 3;
  double dmax = 0.0;
  for (int i = l; i < p; i += 64) dmax = fmax(dmax, A[i * LD + i] + shift);
  for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
  const double delta = 4.0 * EPS * dmax;
  __syncthreads();
  for (int i = threadIdx.x; i < p; i += blockDim.x) A[i * LD + i] += shift + delta;
  __syncthreads();
  (void)chol_lds<PP, true>(p, A, delta);
  // columns scaled by a power of two so that squared norms and their products stay in range
  const double scale = ldexp(1.0, dmax > 0.0 ? -ilogb(dmax) / 2 : 0);
  const bool on = w < nw;
  ColPairs<R> u;
  u.ix = 16 * w + q;
  u.iy = u.ix + 8;
  u.tol = (float)EPS;
  if (on)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = g + 8 * r;
      u.x[r] = row >= u.ix && row < p ? scale * A[row * LD + u.ix] : 0.0;
      u.y[r] = row >= u.iy && row < p ? scale * A[row * LD + u.iy] : 0.0;
    }
  __syncthreads();  // A becomes the exchange buffer
  int sweep = 0;
  for (; sweep < 30; ++sweep) {
    u.cm = u.em = 0.f;
    for (int br = 0; br < 2 * nw - 1; ++br) {
      if (on) u.meet(br == 0);
      if (nw > 1) {
        // circle tournament of the 2 nw blocks: x of wave 0 stays, y of wave 0 -> x of wave 1,
        // x of wave i -> x of wave i + 1, x of the last -> its y, y of wave i -> y of wave i - 1
        __syncthreads();
        if (on) {
          const int tx = w + 1 < nw ? w + 1 : nw + w, ty = w == 0 ? 1 : nw + w - 1;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (w > 0) A[(tx * R + r) * 64 + l] = u.x[r];
            A[(ty * R + r) * 64 + l] = u.y[r];
          }
          if (g == 0) {
            if (w > 0) ids[tx][q] = u.ix;
            ids[ty][q] = u.iy;
          }
        }
        __syncthreads();
        if (on) {
          if (w > 0) u.ix = ids[w][q];
          u.iy = ids[nw + w][q];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (w > 0) u.x[r] = A[(w * R + r) * 64 + l];
            u.y[r] = A[((nw + w) * R + r) * 64 + l];
          }
        }
      }
    }
    float cm = u.cm, em = u.em;
    for (int o = 4; o > 0; o >>= 1) {  // the lane groups hold the same values
      cm = fmaxf(cm, __shfl_xor(cm, o, 64));
      em = fmaxf(em, __shfl_xor(em, o, 64));
    }
    if (on && l == 0) {
      stat[w][0] = cm;
      stat[w][1] = em;
    }
    __syncthreads();
    cm = em = 0.f;
    for (int k = 0; k < nw; ++k) {
      cm = fmaxf(cm, stat[k][0]);
      em = fmaxf(em, stat[k][1]);
    }
    __syncthreads();
    if (!(cm * (em + 4e-7f) > (float)EPS)) break;
  }
  // the columns' directions: U
  if (on) {
    u.norms();
    const double a = u.a, b = u.b;
    const double ra = a > 0.0 ? rsq_nr(a) : 0.0, rb = b > 0.0 ? rsq_nr(b) : 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = g + 8 * r;
      if (row < 16 * nw) {
        const int to = ord[row] * LD;
        A[to + u.ix] = a > 0.0 ? u.x[r] * ra : (row == u.ix ? 1.0 : 0.0);
        A[to + u.iy] = b > 0.0 ? u.y[r] * rb : (row == u.iy ? 1.0 : 0.0);
      }
    }
  }
  return sweep + 1;
}


}  // namespace gsi
