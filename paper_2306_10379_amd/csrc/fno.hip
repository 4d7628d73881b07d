// Sine-basis neural operator for warm starts (see include/fno.h): forward pass, subspace
// loss, gradient and Adam, all as gfx950 kernels on float32 data, with the weights read as
// float32 or from a bfloat16 working copy (Wp).
//
// Data layout: activations channel-major, [sample][channel][N x N grid, row-major], so a
// channel of a sample is one contiguous n = N^2 vector; the network's output Y and the targets
// n x p row-major, as callers hold them. A layer is three kernels: k_sine_fwd (S U S^T of every
// channel, both contractions), k_mix_inv (mixes the channels mode by mode and applies S from one
// side) and k_layer (S from the other side, the pointwise mixing, bias and activation in one pass
// over the grid); the backward pass runs the same three with the weights transposed. Gram-like
// reductions over the whole grid (weight gradients, the p x p Grams of the loss) split the grid over workgroups and add the partial results in a fixed
// order (k_pqt_small, k_gram_rows, k_sum_parts). Contractions are float32 MFMA. The p x p loss
// algebra (Cholesky of Y^T Y) runs in float64, one workgroup per sample.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/fno.h"
#include "gsi_dense_dev.h"
#include "gsi_device.h"

namespace fno {

using gsi::f4;
using gsi::gld;
using gsi::gst;
using gsi::mfma;
constexpr int WG = 256;

__device__ __forceinline__ f4 ld4(const float* p) { return gld(reinterpret_cast<const f4*>(p)); }

// A run of weights: the float32 master, or (h set) its bfloat16 working copy, widened on
// reading. The choice is the same for every thread of a launch.
struct Wp {
  const float* f;
  const uint16_t* h;
  __device__ __forceinline__ float operator[](int64_t i) const {
    return h ? gsi::bf16_widen(gld(h + i)) : gld(f + i);
  }
};

// ---------------------------------------------------------------- sine transform of channels

// H[bc] = S U[bc] S^T, one workgroup of 16 waves per channel. The rows of U stream through once (16
// bytes a lane along a row); S sits in LDS, row stride N + 4 (the 16 rows of an operand load then
// start 4 banks apart), and so does the intermediate U S^T, which the second contraction takes up.
// STAGED: both fit (N <= 608 at 32 modes, always at 16); else S comes from the caches. MFMA operand
// layout: lane (g, c) = (l / 16, l % 16) holds 4 of k at k0 + 4 g of row c, and step q of four
// contracts k0 + 4 g + q over g. Reading U is what the layer cannot do without; two GEMM launches
// with the intermediate in memory, and S read beside U from the caches, took 60 us for 320
// channels of 256 x 256 (84 MB), this 29 us, and 17.5 us for 160 (one a CU, two thirds of it MFMA
// work). Rows are not split over workgroups: the sum over them keeps one order, and few channels
// take no longer than one.
constexpr int SINE_T = 1024;

template <bool STAGED>
__global__ __launch_bounds__(SINE_T) void k_sine_fwd(const float* __restrict__ U, const float* __restrict__ S,
                                                     float* __restrict__ H, int N, int MP) {
  extern __shared__ __align__(16) float lds[];
  const int ld = N + 4, CB = MP / 16, lds_s = STAGED ? ld : N;
  float* sT = lds;  // [k2][row]
  float* sS = lds + MP * ld;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  const int64_t bc = blockIdx.x;
  if constexpr (STAGED) {
    for (int e = threadIdx.x; e < MP * (N / 4); e += SINE_T) {
      const int r = e / (N / 4), q = e - r * (N / 4);
      *reinterpret_cast<f4*>(sS + r * ld + 4 * q) = ld4(S + r * N + 4 * q);
    }
    __syncthreads();
  }
  auto s4 = [&](int r, int k) {
    if constexpr (STAGED) return *reinterpret_cast<const f4*>(sS + r * lds_s + k);
    else return ld4(S + r * lds_s + k);
  };
  const f4 z = {0.f, 0.f, 0.f, 0.f};
  const int c1 = CB > 1 ? 16 + c : c;
  for (int rb = w; rb < N / 16; rb += SINE_T / 64) {
    const float* u = U + (bc * N + 16 * rb + c) * N + 4 * g;
    f4 t0 = z, t1 = z;
#pragma unroll 8
    for (int k0 = 0; k0 < N; k0 += 16) {
      const f4 uv = ld4(u + k0);
      const f4 v0 = s4(c, k0 + 4 * g), v1 = s4(c1, k0 + 4 * g);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        t0 = mfma(uv[q], v0[q], t0);
        t1 = mfma(uv[q], v1[q], t1);
      }
    }
    // rows 4 g .. 4 g + 3 of the block, columns c and 16 + c
    const int at = 16 * rb + 4 * g;
    *reinterpret_cast<f4*>(sT + c * ld + at) = t0;
    if (CB > 1) *reinterpret_cast<f4*>(sT + (16 + c) * ld + at) = t1;
  }
  __syncthreads();
  if (w >= CB * CB) return;
  const int i = w / CB, j = w % CB;
  f4 acc = z;
#pragma unroll 4
  for (int k0 = 0; k0 < N; k0 += 16) {
    const f4 av = s4(16 * i + c, k0 + 4 * g), bv = *reinterpret_cast<const f4*>(sT + (16 * j + c) * ld + k0 + 4 * g);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = mfma(av[q], bv[q], acc);
  }
  float* out = H + bc * MP * MP;
#pragma unroll
  for (int r = 0; r < 4; ++r) gst(out + (16 * i + 4 * g + r) * MP + 16 * j + c, acc[r]);
}

// Output channel `o` of a spectral layer: Vh[b][o][k] = sum_i R_oi[k] H[b][i][k] over the inner
// channels, then Zt[b][o][x][k1] = sum_k2 S[k2][x] Vh[k1][k2], the first half of the inverse
// transform. R_oi = R + (o ro + i ri) m^2. Grid (output channels, samples), a thread per mode: the
// loads of 20 channels are what it waits for (17 us for 16 samples of 20 to 20 channels; separate
// mixing and transform kernels 12 + 17).
template <int MP>
__global__ __launch_bounds__(MP * MP) void k_mix_inv(Wp R, int64_t ro, int64_t ri, const float* __restrict__ H,
                                                     const float* __restrict__ St, float* __restrict__ Zt, int I, int m,
                                                     int N) {
  constexpr int LDV = MP + 4, CB = MP / 16;
  __shared__ __align__(16) float sV[MP * LDV];
  const int o = blockIdx.x, t = threadIdx.x;
  const int64_t b = blockIdx.y, bo = b * gridDim.x + o;
  const int k1 = t / MP, k2 = t % MP;
  float v = 0.f;
  if (k1 < m && k2 < m) {
    const float* h = H + b * I * MP * MP + t;
    const int64_t r = o * ro * m * m + k1 * m + k2;
#pragma unroll 8
    for (int i = 0; i < I; ++i) v += R[r + i * ri * m * m] * gld(h + i * MP * MP);
  }
  sV[k1 * LDV + k2] = v;
  __syncthreads();
  const int w = t >> 6, l = t & 63, g = l >> 4, c = l & 15;
  const f4 z = {0.f, 0.f, 0.f, 0.f};
  f4 va[CB][CB];  // [block of k1][16 of k2]: lane (g, c): row c, k2 = 4 g ..
#pragma unroll
  for (int i = 0; i < CB; ++i)
#pragma unroll
    for (int q = 0; q < CB; ++q) va[i][q] = *reinterpret_cast<const f4*>(sV + (16 * i + c) * LDV + 16 * q + 4 * g);
  for (int xb = w; xb < N / 16; xb += MP * MP / 64) {
    const int64_t x = 16 * xb + c;
    f4 acc[CB];
#pragma unroll
    for (int i = 0; i < CB; ++i) acc[i] = z;
#pragma unroll
    for (int q = 0; q < CB; ++q) {
      const f4 sv = ld4(St + x * MP + 16 * q + 4 * g);
#pragma unroll
      for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i] = mfma(va[i][q][e], sv[e], acc[i]);
    }
    // k1 = 16 i + 4 g .. + 3 of row x
#pragma unroll
    for (int i = 0; i < CB; ++i) gst(reinterpret_cast<f4*>(Zt + (bo * N + x) * MP + 16 * i + 4 * g), acc[i]);
  }
}

// ---------------------------------------------------------------- small outputs, long K

struct PQtSmall {
  const float* P;
  int64_t ldp, sPb;
  const float* Q;
  int64_t ldq, sQb;
  int R, Cc;  // both <= 32
  int64_t K;  // multiple of 16
  int splits;
  float* part;  // [batch][split][PART]
};

// Values of a partial: 32 x 32, then the 32 row sums of P.
constexpr int PART = 1024 + 32;

// Partial P_b Q_b^T, and the row sums of P_b, over the split's share of K: grid (splits, batch).
// Every wave takes every fourth 16-wide step of the share and keeps all four 16 x 16 blocks; the
// waves' sums are added in wave order in LDS. The row sums (a bias gradient beside its weight
// gradient) ride on the rows already loaded: a product with ones, one more MFMA per 16 rows.
__global__ __launch_bounds__(WG) void k_pqt_small(PQtSmall a) {
  __shared__ float red[PART];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  const int s = blockIdx.x, b = blockIdx.y;
  const int64_t nk = a.K / 16;
  const int64_t k_lo = nk * s / a.splits, k_hi = nk * (s + 1) / a.splits;
  const float* P = a.P + (int64_t)b * a.sPb;
  const float* Q = a.Q + (int64_t)b * a.sQb;
  const bool pok0 = c < a.R, pok1 = 16 + c < a.R, qok0 = c < a.Cc, qok1 = 16 + c < a.Cc;
  const float* p0 = P + (pok0 ? c : 0) * a.ldp + 4 * g;
  const float* p1 = P + (pok1 ? 16 + c : 0) * a.ldp + 4 * g;
  const float* q0 = Q + (qok0 ? c : 0) * a.ldq + 4 * g;
  const float* q1 = Q + (qok1 ? 16 + c : 0) * a.ldq + 4 * g;
  const f4 z = {0.f, 0.f, 0.f, 0.f};
  f4 acc[2][2] = {{z, z}, {z, z}}, sum[2] = {z, z};
  constexpr int UN = 4;
  for (int64_t kk = k_lo + w; kk < k_hi; kk += 4 * UN) {
    f4 x[UN][4];  // rows c and 16 + c of P, then of Q
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t k0 = 16 * (kk + 4 * u < k_hi ? kk + 4 * u : kk);
      x[u][0] = ld4(p0 + k0);
      x[u][1] = ld4(p1 + k0);
      x[u][2] = ld4(q0 + k0);
      x[u][3] = ld4(q1 + k0);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const bool in = kk + 4 * u < k_hi;
      const f4 a0 = in && pok0 ? x[u][0] : z, a1 = in && pok1 ? x[u][1] : z;
      const f4 b0 = in && qok0 ? x[u][2] : z, b1 = in && qok1 ? x[u][3] : z;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        sum[0] = mfma(a0[q], 1.f, sum[0]);
        sum[1] = mfma(a1[q], 1.f, sum[1]);
        acc[0][0] = mfma(a0[q], b0[q], acc[0][0]);
        acc[0][1] = mfma(a0[q], b1[q], acc[0][1]);
        acc[1][0] = mfma(a1[q], b0[q], acc[1][0]);
        acc[1][1] = mfma(a1[q], b1[q], acc[1][1]);
      }
    }
  }
  for (int ww = 0; ww < 4; ++ww) {
    if (w == ww) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int e = (16 * rb + 4 * g + r) * 32 + 16 * cb + c;
            red[e] = (ww ? red[e] : 0.f) + acc[rb][cb][r];
          }
      if (c == 0)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int e = 1024 + 16 * rb + 4 * g + r;
            red[e] = (ww ? red[e] : 0.f) + sum[rb][r];
          }
    }
    __syncthreads();
  }
  float* out = a.part + ((int64_t)b * a.splits + s) * PART;
  for (int e = threadIdx.x; e < PART; e += WG) gst(out + e, red[e]);
}

// out[gr][r][c] (at gr so_g + r ldo + c) = the sum of the group's partials, and, with bias given,
// bias[r] = the sum of the row sums. A workgroup takes 16 entries, 16 lanes each a
// share of the partials (16 entries x 4 bytes of a partial are contiguous), and adds the shares
// in a fixed order: one thread per entry, adding up to 512 partials one load after the other on
// two CUs, took 64 us a gradient, 12 times a training step; now 5 us.
constexpr int SUM_E = 16, SUM_S = 16;
template <typename TO>
__global__ __launch_bounds__(SUM_E * SUM_S) void k_sum_parts(const float* part, int per_group, int R, int Cc, TO* out,
                                                             int64_t so_g, int ldo, TO* bias) {
  __shared__ double red[SUM_S][SUM_E];
  const int x = threadIdx.x % SUM_E, q = threadIdx.x / SUM_E, gr = blockIdx.y;
  const int e = blockIdx.x * SUM_E + x;  // rows of 32: the matrix, then the row sums
  const int r = e >> 5, c = e & 31;
  const bool sums = e >= 1024;
  const bool ok = sums ? bias && c < R : r < R && c < Cc;
  double acc = 0.0;
  if (ok) {
    const float* p = part + (int64_t)gr * per_group * PART + e;
#pragma unroll 4
    for (int j = q; j < per_group; j += SUM_S) acc += (double)gld(p + (int64_t)j * PART);
  }
  red[q][x] = acc;
  __syncthreads();
  if (q || !ok) return;
  for (int k = 1; k < SUM_S; ++k) acc += red[k][x];
  if (sums) gst(bias + c, (TO)acc);
  else gst(out + gr * so_g + r * ldo + c, (TO)acc);
}

// ---------------------------------------------------------------- pointwise kernels

__device__ __forceinline__ float gelu(float t) { return 0.5f * t * (1.0f + erff(t * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float t) {
  return 0.5f * (1.0f + erff(t * 0.70710678118654752f)) + t * 0.39894228040143268f * expf(-0.5f * t * t);
}

// In[b] = [V / 20, x, y] (stored when In is given: the weight gradient reads it); U0[b][c] =
// W_lift In + b_lift. Thread per 4 nodes of a row (N is a multiple of 16); vec: V is 16-byte
// aligned.
__global__ __launch_bounds__(WG) void k_lift(const float* V, int N, int w, Wp W, Wp bias, float* In, float* U0, int B,
                                             int vec) {
  __shared__ float sW[32 * 4];
  for (int e = threadIdx.x; e < 4 * w; e += WG) sW[e] = (e & 3) < 3 ? W[3 * (e >> 2) + (e & 3)] : bias[e >> 2];
  __syncthreads();
  const int64_t n = (int64_t)N * N;
  const int64_t id = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (id >= (int64_t)B * n) return;
  const int64_t b = id / n, j = id - b * n;
  const int y = (int)(j / N), x = (int)(j - (int64_t)y * N);
  const float h = 1.0f / (float)(N + 1);
  f4 f0, f1;
  const f4 v = vec ? ld4(V + id) : f4{gld(V + id), gld(V + id + 1), gld(V + id + 2), gld(V + id + 3)};
  const float f2 = (float)(y + 1) * h;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f0[e] = v[e] * 0.05f;
    f1[e] = (float)(x + e + 1) * h;
  }
  if (In) {
    gst(reinterpret_cast<f4*>(In + (b * 3 + 0) * n + j), f0);
    gst(reinterpret_cast<f4*>(In + (b * 3 + 1) * n + j), f1);
    gst(reinterpret_cast<f4*>(In + (b * 3 + 2) * n + j), f4{f2, f2, f2, f2});
  }
  for (int c = 0; c < w; ++c) {
    f4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = sW[4 * c + 3] + sW[4 * c] * f0[e] + sW[4 * c + 1] * f1[e] + sW[4 * c + 2] * f2;
    gst(reinterpret_cast<f4*>(U0 + (b * w + c) * n + j), o);
  }
}

// The rest of a layer on a tile of LY rows x LX nodes, all O output channels:
//   s[o] = sum_k1 S[k1][y] Zt[o][x][k1] + sum_i W_oi U[i] (+ bias[o]),
// W_oi = W[o wo + i wi]. HIDDEN: Pre = s (if given), Out = gelu(s). OUTPUT: s with prior[o] added to
// the bias, row-major n x O into Y32 and / or Y64. BACKWARD: Out = s, times gelu'(Pre) if Pre is
// given (the gradient before the previous layer's activation).
//
// One pass reads U and Zt and writes the result: the second half of the inverse transform has
// its own matrix per channel and the pointwise mixing its own per node, so their MFMA results lie
// differently in the lanes (rows y, columns x of a channel; rows o of 64 nodes) and the first goes
// through LDS (row stride LX + 4: the four lane groups' rows on different banks) to become the
// second's initial accumulator (BACKWARD: to be added to it). In the second, lane c owns the nodes
// 4 c .. 4 c + 3 of its wave's two rows, so that one 16-byte load of a channel feeds four MFMA blocks
// and results leave in 16 bytes.
// Separate kernels with the transform's result in memory and the mixing on the vector unit (a
// broadcast LDS read per weight and node) took 58 + 104 us for 16 samples of 20 x 256 x 256, this
// 67 us (0.17 GB without Pre, 34 us at the copy rate; erff takes about 16 of the rest). The weights
// stay in LDS and the activation runs from the tile: with both in registers the workgroup needed
// 112 VGPRs, two fitted a CU, and it took 78 us; at 80 three fit.
enum { LAYER_HIDDEN, LAYER_OUTPUT, LAYER_BACKWARD };
constexpr int LY = 16, LX = 32, LTX = LX + 4, LDW = 36, LT = 512;

struct Layer {
  const float *Zt, *U, *St;
  Wp W;
  int wo, wi;
  Wp bias;             // HIDDEN, OUTPUT
  const float* prior;  // OUTPUT
  float* Pre;          // HIDDEN: written; BACKWARD: read
  float* Out;          // HIDDEN, BACKWARD
  float* Y32;          // OUTPUT
  double* Y64;
  int vec;             // OUTPUT: O a multiple of 4 and Y32, Y64 16-byte aligned
  int O, I, N, MP;
};

template <int MODE, int OB>
__global__ __launch_bounds__(LT, MODE == LAYER_OUTPUT ? 4 : 6) void k_layer(Layer a) {
  extern __shared__ __align__(16) float lds[];
  float* sW = lds;  // [16 OB][LDW], the bias
  float* tile = lds + 16 * OB * (LDW + 1);  // [o][LY][LTX]
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  const int N = a.N, MP = a.MP, O = a.O, I = a.I;
  const int x0 = blockIdx.x * LX, y0 = blockIdx.y * LY;
  const int64_t b = blockIdx.z, n = (int64_t)N * N;
  const f4 z = {0.f, 0.f, 0.f, 0.f};
  // this lane's nodes: row y0 + 2 w + c / 8, columns x0 + 4 (c mod 8) ..
  const int xc = 4 * (c & 7), ty = 2 * w + (c >> 3);
  const bool xok = x0 + xc < N;
  const int64_t nd = (int64_t)(y0 + ty) * N + x0 + (xok ? xc : 0);
  constexpr int KS = 8;  // at most 32 inner channels, 4 a step
  f4 u[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    u[s] = z;
    if (4 * s >= I) continue;
    const f4 v = ld4(a.U + (b * I + min(4 * s + g, I - 1)) * n + nd);
    if (4 * s + g < I) u[s] = v;
  }
  float* sB = sW + 16 * OB * LDW;
  for (int e = threadIdx.x; e < 16 * OB * 32; e += LT) {
    const int o = e >> 5, i = e & 31;
    sW[o * LDW + i] = o < O && i < I ? a.W[o * a.wo + i * a.wi] : 0.f;
  }
  if (threadIdx.x < 16 * OB) sB[threadIdx.x] = MODE != LAYER_BACKWARD && threadIdx.x < O ? a.bias[threadIdx.x] : 0.f;
  // spectral part: wave w takes the column block w & 1 of every fourth channel
  {
    const int xb = w & 1;
    if (x0 + 16 * xb < N) {
      const float* sy = a.St + (int64_t)(y0 + c) * MP + 4 * g;
      const f4 s0 = ld4(sy), s1 = MP > 16 ? ld4(sy + 16) : z;
      const float* zp = a.Zt + (b * O * N + x0 + 16 * xb + c) * MP + 4 * g;
#pragma unroll 4
      for (int o = w >> 1; o < O; o += LT / 128) {
        const float* q0 = zp + (int64_t)o * N * MP;
        const f4 z0 = ld4(q0), z1 = MP > 16 ? ld4(q0 + 16) : z;
        f4 acc = z;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = mfma(s0[q], z0[q], acc);
        if (MP > 16)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc = mfma(s1[q], z1[q], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) tile[(o * LY + 4 * g + r) * LTX + 16 * xb + c] = acc[r];
      }
    }
  }
  __syncthreads();
  f4 acc[OB][4];  // [block of o][node]: register r is channel 16 ob + 4 g + r
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) {
    const f4 bias = *reinterpret_cast<const f4*>(sB + 16 * ob + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 16 * ob + 4 * g + r;
      const int on = min(o, O - 1);  // rows from O on are not used
      f4 t = z;
      if (MODE != LAYER_BACKWARD) t = *reinterpret_cast<const f4*>(tile + (on * LY + ty) * LTX + xc);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[ob][q][r] = t[q] + bias[r];
      if (MODE == LAYER_OUTPUT) {
        const f4 pr = ld4(a.prior + on * n + nd);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[ob][q][r] += pr[q];
      }
    }
  }
#pragma unroll
  for (int s = 0; s < KS; ++s)
    if (4 * s < I)
#pragma unroll
      for (int ob = 0; ob < OB; ++ob) {
        const float wv = sW[(16 * ob + c) * LDW + 4 * s + g];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[ob][q] = mfma(wv, u[s][q], acc[ob][q]);
      }
  if constexpr (MODE == LAYER_OUTPUT) {
    if (!xok) return;
#pragma unroll
    for (int ob = 0; ob < OB; ++ob) {
      const int o0 = 16 * ob + 4 * g;
      if (o0 >= O) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t at = (b * n + nd + q) * O + o0;
        if (a.vec) {
          if (a.Y32) gst(reinterpret_cast<f4*>(a.Y32 + at), acc[ob][q]);
          if (a.Y64) {
            gst(reinterpret_cast<gsi::d2*>(a.Y64 + at), gsi::d2{acc[ob][q][0], acc[ob][q][1]});
            gst(reinterpret_cast<gsi::d2*>(a.Y64 + at + 2), gsi::d2{acc[ob][q][2], acc[ob][q][3]});
          }
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (o0 + r < O) {
              if (a.Y32) gst(a.Y32 + at + r, acc[ob][q][r]);
              if (a.Y64) gst(a.Y64 + at + r, (double)acc[ob][q][r]);
            }
        }
      }
    }
  } else {
    // back to the tile: the activation then takes 4 nodes of a channel a thread, also where O is
    // no multiple of 16, in a loop that needs few registers
#pragma unroll
    for (int ob = 0; ob < OB; ++ob)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = 16 * ob + 4 * g + r;
        if (o >= O || !xok) continue;
        f4* slot = reinterpret_cast<f4*>(tile + (o * LY + ty) * LTX + xc);
        f4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = acc[ob][q][r];
        if (MODE == LAYER_BACKWARD) v += *slot;
        *slot = v;
      }
    __syncthreads();
    const int row = (threadIdx.x >> 3) & 15, col = 4 * (threadIdx.x & 7);
    if (x0 + col >= N) return;
    const int64_t at = b * O * n + (int64_t)(y0 + row) * N + x0 + col;
#pragma unroll 1
    for (int o = threadIdx.x >> 7; o < O; o += LT / 128) {
      f4 v = *reinterpret_cast<const f4*>(tile + (o * LY + row) * LTX + col);
      if constexpr (MODE == LAYER_HIDDEN) {
        if (a.Pre) gst(reinterpret_cast<f4*>(a.Pre + at + o * n), v);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = gelu(v[q]);
      } else if (a.Pre) {
        const f4 pre = ld4(a.Pre + at + o * n);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] *= gelu_d(pre[q]);
      }
      gst(reinterpret_cast<f4*>(a.Out + at + o * n), v);
    }
  }
}

// ---------------------------------------------------------------- mode-wise weight gradient

// dR[o][c][k1][k2] = sum_b dVh[b][o][k] Uh[b][c][k].
__global__ void k_mix_wgrad(const float* dVh, const float* Uh, float* dR, int B, int O, int C, int m, int MP) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)O * C * m * m) return;
  const int64_t oc = id / (m * m), k = id % (m * m);
  const int k1 = (int)(k / m), k2 = (int)(k % m);
  const int64_t o = oc / C, c = oc % C;
  const int64_t per = (int64_t)MP * MP, kp = (int64_t)k1 * MP + k2;
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += gld(dVh + ((int64_t)b * O + o) * per + kp) * gld(Uh + ((int64_t)b * C + c) * per + kp);
  gst(dR + id, s);
}

// ---------------------------------------------------------------- loss

// One workgroup per sample: G = Y^T Y, Bm = X*^T Y (float64, rows of 32). Cholesky of G = L L^T,
// with Li = L^-1, F = Bm Li^T: loss = p - |F|_F^2, and the coefficients of the gradient
// dLoss/dY = scale (Y Kc - X* Ec) with Ec = Bm G^-1 = F Li and Kc = Ec^T Ec, scale = 2 / batch,
// stored transposed (Kt, Et). The
// factorization and the products are the p x p routines of the eigensolver (float64 MFMA): a
// serial Cholesky by one thread took 550 us.
__global__ __launch_bounds__(WG) void k_loss_small(const double* G, const double* Bm, int p, double scale,
                                                   double* loss, float* Kt, float* Et, int* bad) {
  constexpr int PP = 32, NB = PP / 16, LD = gsi::DLD<PP>;
  __shared__ double L[PP * LD], M[PP * LD], Bs[PP * LD], F[PP * LD], E[PP * LD];
  __shared__ double part[WG / 64];
  __shared__ int sbad;
  const int b = blockIdx.x, t = threadIdx.x, nb = (p + 15) >> 4, m = 16 * nb;
  const double* Gb = G + (int64_t)b * 1024;
  const double* Bb = Bm + (int64_t)b * 1024;
  gsi::fill_dense(m, L, LD, [&](int i, int j) { return i < p && j < p ? 0.5 * (Gb[i * 32 + j] + Gb[j * 32 + i]) : 0.0; });
  gsi::fill_dense(m, Bs, LD, [&](int i, int j) { return i < p && j < p ? Bb[i * 32 + j] : 0.0; });
  __syncthreads();
  const bool low = gsi::chol_lds<PP, false>(p, L, 0.0);
  if (t == 0) sbad = low;
  __syncthreads();
  float* Kb = Kt + (int64_t)b * 1024;
  float* Eb = Et + (int64_t)b * 1024;
  for (int e = t; e < 1024; e += WG) Kb[e] = Eb[e] = 0.f;
  if (sbad) {
    if (t == 0) { loss[b] = NAN; atomicExch(bad, 1); }
    return;
  }
  gsi::inv_chol<PP>(p, L, M, LD);  // M = Li^T
  __syncthreads();
  gsi::mm_dense<NB, LD, false, LD, false>(nb, Bs, M, [&](int i, int j, double v) { F[i * LD + j] = v; });
  __syncthreads();
  gsi::mm_dense<NB, LD, false, LD, true>(nb, F, M, [&](int i, int j, double v) {
    E[i * LD + j] = v;
    Eb[j * 32 + i] = (float)(scale * v);
  });
  double s = 0.0;
  for (int e = t; e < m * m; e += WG) {
    const double f = F[e / m * LD + e % m];
    s = fma(f, f, s);
  }
  s = gsi::wave_sum(s);
  if ((t & 63) == 0) part[t >> 6] = s;
  __syncthreads();
  if (t == 0) loss[b] = (double)p - (((part[0] + part[1]) + part[2]) + part[3]);
  gsi::mm_dense<NB, LD, true, LD, false>(nb, E, E, [&](int i, int j, double v) { Kb[j * 32 + i] = (float)(scale * v); });
}

// Partial G = Y^T Y and Bm = X^T Y of sample blockIdx.y over the split's rows, Y and X n x p
// row-major: lane (g, c) holds rows 4 g .. 4 g + 3 of a step, column 16 cb + c, both operands'
// layout (the rows of a step share their cache lines over q). Partials of G in part, of Bm after
// those of all samples.
__global__ __launch_bounds__(WG) void k_gram_rows(const float* __restrict__ Y, const float* __restrict__ X, int p,
                                                  int64_t n, int splits, float* __restrict__ part) {
  __shared__ float red[2 * 1024];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  const int s = blockIdx.x, b = blockIdx.y;
  const int64_t nk = n / 16, k_lo = nk * s / splits, k_hi = nk * (s + 1) / splits;
  const float* Yb = Y + (int64_t)b * n * p;
  const float* Xb = X + (int64_t)b * n * p;
  const bool ok0 = c < p, ok1 = 16 + c < p;
  const f4 z = {0.f, 0.f, 0.f, 0.f};
  f4 G[2][2] = {{z, z}, {z, z}}, M[2][2] = {{z, z}, {z, z}};
  const int c0 = ok0 ? c : 0, c1 = ok1 ? 16 + c : 0;  // a column to load in any case
  constexpr int UN = 2;
  for (int64_t kk = k_lo + w; kk < k_hi; kk += 4 * UN) {
    float v[UN][4][4];  // columns c and 16 + c of Y, then of X
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t o = ((kk + 4 * u < k_hi ? kk + 4 * u : kk) * 16 + 4 * g + q) * p;
        v[u][0][q] = gld(Yb + o + c0);
        v[u][1][q] = gld(Yb + o + c1);
        v[u][2][q] = gld(Xb + o + c0);
        v[u][3][q] = gld(Xb + o + c1);
      }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const bool in = kk + 4 * u < k_hi;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float y[2] = {in && ok0 ? v[u][0][q] : 0.f, in && ok1 ? v[u][1][q] : 0.f};
        const float x[2] = {in && ok0 ? v[u][2][q] : 0.f, in && ok1 ? v[u][3][q] : 0.f};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            G[i][j] = mfma(y[i], y[j], G[i][j]);
            M[i][j] = mfma(x[i], y[j], M[i][j]);
          }
      }
    }
  }
  for (int ww = 0; ww < 4; ++ww) {
    if (w == ww) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int e = (16 * i + 4 * g + r) * 32 + 16 * j + c;
            red[e] = (ww ? red[e] : 0.f) + G[i][j][r];
            red[1024 + e] = (ww ? red[1024 + e] : 0.f) + M[i][j][r];
          }
    }
    __syncthreads();
  }
  float* o0 = part + ((int64_t)b * splits + s) * PART;
  float* o1 = o0 + (int64_t)gridDim.y * splits * PART;
  for (int e = threadIdx.x; e < 1024; e += WG) {
    gst(o0 + e, red[e]);
    gst(o1 + e, red[1024 + e]);
  }
}

// dY[b][a][i] = sum_q Y[b][i][q] Kt[a][q] - X[b][i][q] Et[a][q]: Y and X row-major, dY
// channel-major. Thread per node: its two rows in registers (16-byte loads when vec: p a multiple
// of 4, X 16-byte aligned), the coefficients wave-uniform through the scalar cache. The terms of a
// q cancel to a large part (the gradient is what of X lies off span(Y)), so each is rounded by
// itself before it is added; a chain over all products, as the matrix cores form it, is not the
// same sum. 69 us for 8 samples of 65536 x 32 (0.2 GB); with X copied to channel-major first and
// the coefficients broadcast from LDS 181 us.
__global__ __launch_bounds__(WG) void k_loss_dy(const float* __restrict__ Y, const float* __restrict__ X,
                                                const float* __restrict__ Kt, const float* __restrict__ Et,
                                                float* __restrict__ dY, int p, int64_t n, int vec) {
  const int64_t b = blockIdx.y, i = (int64_t)blockIdx.x * WG + threadIdx.x;  // n is a multiple of WG
  const float* ys = Y + (b * n + i) * p;
  const float* xs = X + (b * n + i) * p;
  float y[32], x[32];
  if (vec) {
#pragma unroll
    for (int q = 0; q < 32; q += 4) {
      const f4 z = {0.f, 0.f, 0.f, 0.f};
      const f4 yv = q < p ? ld4(ys + q) : z, xv = q < p ? ld4(xs + q) : z;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[q + e] = yv[e];
        x[q + e] = xv[e];
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      y[q] = q < p ? gld(ys + q) : 0.f;
      x[q] = q < p ? gld(xs + q) : 0.f;
    }
  }
  for (int a = 0; a < p; ++a) {
    const float* k = Kt + b * 1024 + a * 32;
    const float* e = Et + b * 1024 + a * 32;
    float s = 0.f;
#pragma unroll
    for (int h = 0; h < 32; h += 16)  // zeros beyond p
      if (h < p)
#pragma unroll
        for (int q = h; q < h + 16; ++q) s += fmaf(k[q], y[q], -(e[q] * x[q]));
    gst(dY + (b * p + a) * n + i, s);
  }
}

// ---------------------------------------------------------------- Adam

// Adam on the float32 master w; wbf (nullable) receives the updated weights rounded to bfloat16.
__global__ void k_adam(float* w, uint16_t* wbf, const float* g, float* m1, float* m2, int64_t count, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = gld(g + i);
  const float m = b1 * gld(m1 + i) + (1.f - b1) * gi;
  const float v = b2 * gld(m2 + i) + (1.f - b2) * gi * gi;
  gst(m1 + i, m);
  gst(m2 + i, v);
  const float nw = gld(w + i) - lr * (m / c1) / (sqrtf(v / c2) + eps);
  gst(w + i, nw);
  if (wbf) gst(wbf + i, gsi::bf16_round(nw));
}

__global__ void k_round_bf16(const float* w, uint16_t* wbf, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) gst(wbf + i, gsi::bf16_round(gld(w + i)));
}

// splitmix64 (Steele, Lea, Flood 2014) and Box-Muller for the seeded initial weights.
struct Rng {
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  double uniform() { return ((next() >> 11) + 0.5) * (1.0 / 9007199254740992.0); }
  double normal() { return sqrt(-2.0 * log(uniform())) * cos(6.283185307179586 * uniform()); }
};

}  // namespace fno

using namespace fno;

struct fno_net {
  fno_config cfg{};
  int MP = 0;
  int64_t n = 0, count = 0;
  hipStream_t st = nullptr;
  bool own_stream = false;
  std::string err;
  std::vector<void*> allocs;
  // parameter offsets: lift, per hidden layer (R, W, b), output layer (R, W, b)
  int64_t oWl = 0, obl = 0;
  std::vector<int64_t> oR, oW, ob;  // L + 1 entries, the last is the output layer
  float *params = nullptr, *grad = nullptr, *m1 = nullptr, *m2 = nullptr;
  uint16_t* wbf = nullptr;  // bfloat16 working copy of params (bf16_weights), else null
  int64_t step = 0;
  float *S = nullptr, *St = nullptr, *prior = nullptr;
  float *In = nullptr, *Y = nullptr, *dY = nullptr, *dPa = nullptr, *dPb = nullptr;
  float *dVh = nullptr, *Zt = nullptr, *part = nullptr;
  std::vector<float*> act, pre, uh;
  double *G = nullptr, *Bm = nullptr, *lossd = nullptr;
  float *Kt = nullptr, *Et = nullptr;
  int* bad = nullptr;
  int splits = 1;
};

namespace {

bool valid(const fno_config* c) {
  return c && c->N >= 16 && c->N <= 1024 && c->N % 16 == 0 && c->modes >= 1 && c->modes <= 32 && c->modes <= c->N &&
         c->width >= 1 && c->width <= 32 && c->p >= 1 && c->p <= 32 && c->layers >= 0 && c->max_batch >= 1 &&
         (c->bf16_weights == 0 || c->bf16_weights == 1);
}

// The weights at parameter offset off, in the format the passes read.
Wp wp(const fno_net* h, int64_t off) { return Wp{h->params + off, h->wbf ? h->wbf + off : nullptr}; }

int64_t count_params(const fno_config* c) {
  const int64_t w = c->width, m = c->modes, p = c->p;
  return 3 * w + w + c->layers * (w * w * m * m + w * w + w) + p * w * m * m + p * w + p;
}

template <typename U>
U* nalloc(fno_net* h, size_t count, hipError_t& e) {
  void* ptr = nullptr;
  if (e != hipSuccess) return nullptr;
  e = hipMalloc(&ptr, std::max<size_t>(count, 1) * sizeof(U) + 256);
  if (e != hipSuccess) return nullptr;
  h->allocs.push_back(ptr);
  return reinterpret_cast<U*>(ptr);
}

constexpr size_t LDS_MAX = 160 * 1024;  // of a workgroup

inline unsigned blocks(int64_t work, int per = WG) { return (unsigned)((work + per - 1) / per); }

// H = S U[bc] S^T for BC channels
void sine_fwd(fno_net* h, const float* U, int BC, float* H) {
  const int N = h->cfg.N, MP = h->MP;
  const size_t half = sizeof(float) * MP * (N + 4);
  if (2 * half <= LDS_MAX) k_sine_fwd<true><<<BC, SINE_T, 2 * half, h->st>>>(U, h->S, H, N, MP);
  else k_sine_fwd<false><<<BC, SINE_T, half, h->st>>>(U, h->S, H, N, MP);
}

// Zt[b][o] from I inner channels H and the spectral weights at offset oR (element (o, i) at
// (o ro + i ri) m^2)
void mix_inv(fno_net* h, int64_t oR, int64_t ro, int64_t ri, const float* H, int O, int I, int B) {
  auto go = [&](auto* k) {
    k<<<dim3(O, B), h->MP * h->MP, 0, h->st>>>(wp(h, oR), ro, ri, H, h->St, h->Zt, I, h->cfg.modes, h->cfg.N);
  };
  if (h->MP == 16) go(k_mix_inv<16>);
  else go(k_mix_inv<32>);
}

template <int MODE>
void layer(fno_net* h, Layer a, int B) {
  a.Zt = h->Zt;
  a.St = h->St;
  a.N = h->cfg.N;
  a.MP = h->MP;
  const dim3 grid((a.N + LX - 1) / LX, a.N / LY, B);
  const int ob = a.O <= 16 ? 1 : 2;
  const size_t lds = sizeof(float) * (16 * ob * (LDW + 1) + a.O * LY * LTX);
  if (ob == 1) k_layer<MODE, 1><<<grid, LT, lds, h->st>>>(a);
  else k_layer<MODE, 2><<<grid, LT, lds, h->st>>>(a);
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

// out (R x Cc, row stride Cc) = the sum over the batch of P_b Q_b^T, with P_b: R x n, Q_b: Cc x n;
// bias: the row sums of P over the batch.
void gram_small(fno_net* h, const float* P, const float* Q, int R, int Cc, int B, float* out, float* bias) {
  PQtSmall a{P, h->n, R * h->n, Q, h->n, Cc * h->n, R, Cc, h->n, h->splits, h->part};
  k_pqt_small<<<dim3((unsigned)h->splits, (unsigned)B), WG, 0, h->st>>>(a);
  k_sum_parts<float><<<PART / SUM_E, SUM_E * SUM_S, 0, h->st>>>(h->part, B * h->splits, R, Cc, out, 0, Cc, bias);
}

// Forward pass into Y32 / Y64 (row-major, nullable); train: keeps what the backward pass reads.
void forward(fno_net* h, const float* V, int B, float* Y32, double* Y64, bool train) {
  const fno_config& c = h->cfg;
  const int w = c.width, p = c.p, L = c.layers;
  k_lift<<<blocks(B * h->n / 4), WG, 0, h->st>>>(V, c.N, w, wp(h, h->oWl), wp(h, h->obl), train ? h->In : nullptr,
                                                 h->act[0], B, aligned16(V) ? 1 : 0);
  for (int l = 0; l <= L; ++l) {
    const int O = l < L ? w : p;
    sine_fwd(h, h->act[l], B * w, h->uh[l]);
    mix_inv(h, h->oR[l], w, 1, h->uh[l], O, w, B);
    Layer a{};
    a.U = h->act[l];
    a.W = wp(h, h->oW[l]);
    a.wo = w;
    a.wi = 1;
    a.bias = wp(h, h->ob[l]);
    a.O = O;
    a.I = w;
    if (l < L) {
      a.Pre = train ? h->pre[l] : nullptr;
      a.Out = h->act[l + 1];
      layer<LAYER_HIDDEN>(h, a, B);
    } else {
      a.prior = h->prior;
      a.Y32 = Y32;
      a.Y64 = Y64;
      a.vec = p % 4 == 0 && aligned16(Y32) && aligned16(Y64);
      layer<LAYER_OUTPUT>(h, a, B);
    }
  }
}

// Backward from dY (channel-major, the gradient of the mean loss) into h->grad.
void backward(fno_net* h, int B) {
  const fno_config& c = h->cfg;
  const int w = c.width, p = c.p, L = c.layers, m = c.modes;
  const float* dP = h->dY;  // gradient before layer l's activation
  float *cur = h->dPa, *nxt = h->dPb;
  for (int l = L; l >= 0; --l) {
    const int O = l < L ? w : p;
    // W and b gradients: sums over samples and nodes
    gram_small(h, dP, h->act[l], O, w, B, h->grad + h->oW[l], h->grad + h->ob[l]);
    // spectral part: dVh = S dP S^T, dR; then dU = W^T dP + S^T dUh S, and the previous layer's
    // activation
    sine_fwd(h, dP, B * O, h->dVh);
    mix_inv(h, h->oR[l], 1, w, h->dVh, w, O, B);
    k_mix_wgrad<<<blocks((int64_t)O * w * m * m), WG, 0, h->st>>>(h->dVh, h->uh[l], h->grad + h->oR[l], B, O, w, m, h->MP);
    Layer a{};
    a.U = dP;
    a.W = wp(h, h->oW[l]);
    a.wo = 1;
    a.wi = w;
    a.Pre = l > 0 ? h->pre[l - 1] : nullptr;
    a.Out = cur;
    a.O = w;
    a.I = O;
    layer<LAYER_BACKWARD>(h, a, B);
    dP = cur;
    std::swap(cur, nxt);
  }
  // lift: dP is dU_0
  gram_small(h, dP, h->In, w, 3, B, h->grad + h->oWl, h->grad + h->obl);
}

gsi_status hip_status(fno_net* h, hipError_t e, const char* what) {
  if (e == hipSuccess) return GSI_OK;
  h->err = std::string(what) + ": " + hipGetErrorString(e);
  return GSI_EDEVICE;
}

}  // namespace

extern "C" {

int64_t fno_param_count(const fno_config* cfg) { return valid(cfg) ? count_params(cfg) : -1; }

gsi_status fno_create(fno_handle* out, const fno_config* cfg, uint64_t seed, void* stream) {
  if (!out) return GSI_EINVAL;
  *out = nullptr;
  fno_net* h = new (std::nothrow) fno_net();
  if (!h) return GSI_ENOMEM;
  *out = h;
  if (!valid(cfg)) {
    h->err = "invalid configuration (N a multiple of 16 in 16..1024, 1 <= modes <= 32, width, p <= 32, bf16_weights 0 or 1)";
    return GSI_EINVAL;
  }
  h->cfg = *cfg;
  const fno_config& c = h->cfg;
  h->MP = (c.modes + 15) / 16 * 16;
  h->n = (int64_t)c.N * c.N;
  h->count = count_params(cfg);
  h->splits = (int)std::max<int64_t>(1, std::min<int64_t>(32, h->n / 16 / 16));
  h->st = reinterpret_cast<hipStream_t>(stream);
  if (!h->st) {
    if (hipStreamCreate(&h->st) != hipSuccess) { h->err = "stream creation failed"; return GSI_EDEVICE; }
    h->own_stream = true;
  }
  const int w = c.width, p = c.p, L = c.layers, m = c.modes, N = c.N, MP = h->MP;
  const int64_t n = h->n, B = c.max_batch, mx = std::max(w, p);
  // parameter offsets in the documented order
  int64_t off = 0;
  h->oWl = off; off += 3 * w;
  h->obl = off; off += w;
  for (int l = 0; l <= L; ++l) {
    const int64_t O = l < L ? w : p;
    h->oR.push_back(off); off += O * w * m * m;
    h->oW.push_back(off); off += O * w;
    h->ob.push_back(off); off += O;
  }
  hipError_t e = hipSuccess;
  h->params = nalloc<float>(h, h->count, e);
  h->grad = nalloc<float>(h, h->count, e);
  if (c.bf16_weights) h->wbf = nalloc<uint16_t>(h, h->count, e);
  h->m1 = nalloc<float>(h, h->count, e);
  h->m2 = nalloc<float>(h, h->count, e);
  h->S = nalloc<float>(h, (size_t)MP * N, e);
  h->St = nalloc<float>(h, (size_t)N * MP, e);
  h->prior = nalloc<float>(h, (size_t)p * n, e);
  h->In = nalloc<float>(h, B * 3 * n, e);
  for (int l = 0; l <= L; ++l) h->act.push_back(nalloc<float>(h, B * w * n, e));
  for (int l = 0; l < L; ++l) h->pre.push_back(nalloc<float>(h, B * w * n, e));
  for (int l = 0; l <= L; ++l) h->uh.push_back(nalloc<float>(h, B * w * MP * MP, e));
  h->Y = nalloc<float>(h, B * p * n, e);
  h->dY = nalloc<float>(h, B * p * n, e);
  h->dPa = nalloc<float>(h, B * w * n, e);
  h->dPb = nalloc<float>(h, B * w * n, e);
  h->Zt = nalloc<float>(h, B * mx * N * MP, e);
  h->dVh = nalloc<float>(h, B * mx * MP * MP, e);
  h->part = nalloc<float>(h, (size_t)2 * B * h->splits * PART, e);
  h->G = nalloc<double>(h, B * 1024, e);
  h->Bm = nalloc<double>(h, B * 1024, e);
  h->lossd = nalloc<double>(h, B, e);
  h->Kt = nalloc<float>(h, B * 1024, e);
  h->Et = nalloc<float>(h, B * 1024, e);
  h->bad = nalloc<int>(h, 1, e);
  if (e != hipSuccess) { h->err = "out of device memory"; return GSI_ENOMEM; }
  // dynamic LDS above the default limit
  for (const void* k : {reinterpret_cast<const void*>(k_sine_fwd<true>),
                        reinterpret_cast<const void*>(k_sine_fwd<false>),
                        reinterpret_cast<const void*>(k_layer<LAYER_HIDDEN, 2>),
                        reinterpret_cast<const void*>(k_layer<LAYER_OUTPUT, 2>),
                        reinterpret_cast<const void*>(k_layer<LAYER_BACKWARD, 2>)})
    if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX);
  if (e != hipSuccess) return hip_status(h, e, "kernel attributes");
  // host-side constants: sine matrices (zero beyond m), seeded parameters
  std::vector<float> S((size_t)MP * N, 0.f), St((size_t)N * MP, 0.f), prm(h->count, 0.f);
  const double sc = sqrt(2.0 / (N + 1));
  for (int k = 0; k < m; ++k)
    for (int i = 0; i < N; ++i) {
      const double v = sc * sin(M_PI * (double)(k + 1) * (double)(i + 1) / (double)(N + 1));
      S[(size_t)k * N + i] = (float)v;
      St[(size_t)i * MP + k] = (float)v;
    }
  // prior: sqrt(n) times the p lowest Dirichlet modes s_l(row) s_k(col), by k^2 + l^2, then k
  std::vector<float> prior((size_t)p * n);
  {
    std::vector<std::pair<int, int>> modes;
    const int K = (int)ceil(sqrt(2.0 * p)) + 2;
    for (int k = 1; k <= K; ++k)
      for (int l = 1; l <= K; ++l) modes.push_back({k, l});
    std::stable_sort(modes.begin(), modes.end(), [](const std::pair<int, int>& x, const std::pair<int, int>& y) {
      const int ex = x.first * x.first + x.second * x.second, ey = y.first * y.first + y.second * y.second;
      return ex != ey ? ex < ey : x.first < y.first;
    });
    for (int a = 0; a < p; ++a) {
      const int k = modes[a].first, l = modes[a].second;
      for (int r = 0; r < N; ++r)
        for (int c2 = 0; c2 < N; ++c2)
          prior[(size_t)a * n + (size_t)r * N + c2] =
              (float)((double)N * sc * sin(M_PI * l * (r + 1.0) / (N + 1.0)) * sc * sin(M_PI * k * (c2 + 1.0) / (N + 1.0)));
    }
  }
  Rng rng{seed};
  auto fill = [&](int64_t o, int64_t cnt, double sd) {
    for (int64_t i = 0; i < cnt; ++i) prm[o + i] = (float)(sd * rng.normal());
  };
  fill(h->oWl, 3 * w, 1.0 / sqrt(3.0));
  for (int l = 0; l < L; ++l) {  // the output layer starts at zero: the network starts at the prior
    fill(h->oR[l], (int64_t)w * w * m * m, 1.0 / sqrt((double)w));
    fill(h->oW[l], (int64_t)w * w, 1.0 / sqrt((double)w));
  }
  e = hipMemcpyAsync(h->S, S.data(), S.size() * 4, hipMemcpyHostToDevice, h->st);
  if (e == hipSuccess) e = hipMemcpyAsync(h->St, St.data(), St.size() * 4, hipMemcpyHostToDevice, h->st);
  if (e == hipSuccess) e = hipMemcpyAsync(h->params, prm.data(), prm.size() * 4, hipMemcpyHostToDevice, h->st);
  if (e == hipSuccess) e = hipMemcpyAsync(h->prior, prior.data(), prior.size() * 4, hipMemcpyHostToDevice, h->st);
  if (e == hipSuccess) e = hipMemsetAsync(h->m1, 0, h->count * 4, h->st);
  if (e == hipSuccess) e = hipMemsetAsync(h->m2, 0, h->count * 4, h->st);
  if (e == hipSuccess) e = hipMemsetAsync(h->grad, 0, h->count * 4, h->st);
  if (e == hipSuccess && h->wbf) {
    k_round_bf16<<<blocks(h->count), WG, 0, h->st>>>(h->params, h->wbf, h->count);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(h->st);
  return hip_status(h, e, "create");
}

void* fno_stream(fno_handle h) { return h ? h->st : nullptr; }

gsi_status fno_set_params(fno_handle h, const float* params) {
  if (!h || !params) return GSI_EINVAL;
  hipError_t e = hipMemcpyAsync(h->params, params, h->count * 4, hipMemcpyDeviceToDevice, h->st);
  if (e == hipSuccess && h->wbf) {
    k_round_bf16<<<blocks(h->count), WG, 0, h->st>>>(h->params, h->wbf, h->count);
    e = hipGetLastError();
  }
  return hip_status(h, e, "set_params");
}

gsi_status fno_get_params(fno_handle h, float* params) {
  if (!h || !params) return GSI_EINVAL;
  hipError_t e = hipMemcpyAsync(params, h->params, h->count * 4, hipMemcpyDeviceToDevice, h->st);
  if (e == hipSuccess) e = hipStreamSynchronize(h->st);
  return hip_status(h, e, "get_params");
}

gsi_status fno_forward(fno_handle h, const float* V, int32_t B, float* Y32, double* Y64) {
  if (!h || !V || B < 1 || B > h->cfg.max_batch) return GSI_EINVAL;
  forward(h, V, B, Y32, Y64, false);
  return hip_status(h, hipGetLastError(), "forward");
}

gsi_status fno_loss_grad(fno_handle h, const float* V, const float* Xs, int32_t B, double* loss, float* grad) {
  if (!h || !V || !Xs || B < 1 || B > h->cfg.max_batch) return GSI_EINVAL;
  const int p = h->cfg.p;
  const int64_t n = h->n;
  forward(h, V, B, h->Y, nullptr, true);
  hipError_t e = hipMemsetAsync(h->bad, 0, sizeof(int), h->st);
  k_gram_rows<<<dim3((unsigned)h->splits, (unsigned)B), WG, 0, h->st>>>(h->Y, Xs, p, n, h->splits, h->part);
  for (int q = 0; q < 2; ++q)
    k_sum_parts<double><<<dim3(32 * p / SUM_E, (unsigned)B), SUM_E * SUM_S, 0, h->st>>>(
        h->part + (int64_t)q * B * h->splits * PART, h->splits, p, p, q ? h->Bm : h->G, 1024, 32, nullptr);
  k_loss_small<<<B, WG, 0, h->st>>>(h->G, h->Bm, p, 2.0 / B, h->lossd, h->Kt, h->Et, h->bad);
  k_loss_dy<<<dim3((unsigned)(n / WG), (unsigned)B), WG, 0, h->st>>>(
      h->Y, Xs, h->Kt, h->Et, h->dY, p, n, p % 4 == 0 && aligned16(Xs) ? 1 : 0);
  backward(h, B);
  if (e == hipSuccess && grad) e = hipMemcpyAsync(grad, h->grad, h->count * 4, hipMemcpyDeviceToDevice, h->st);
  std::vector<double> lh(B);
  int bad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(lh.data(), h->lossd, B * sizeof(double), hipMemcpyDeviceToHost, h->st);
  if (e == hipSuccess) e = hipMemcpyAsync(&bad, h->bad, sizeof(int), hipMemcpyDeviceToHost, h->st);
  if (e == hipSuccess) e = hipStreamSynchronize(h->st);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) return hip_status(h, e, "loss_grad");
  if (loss)
    for (int i = 0; i < B; ++i) loss[i] = lh[i];
  if (bad) { h->err = "singular Gram Y^T Y in the loss"; return GSI_EDEVICE; }
  return GSI_OK;
}

gsi_status fno_adam(fno_handle h, float lr, float beta1, float beta2, float eps) {
  if (!h) return GSI_EINVAL;
  ++h->step;
  const float c1 = 1.f - powf(beta1, (float)h->step), c2 = 1.f - powf(beta2, (float)h->step);
  k_adam<<<blocks(h->count), WG, 0, h->st>>>(h->params, h->wbf, h->grad, h->m1, h->m2, h->count, lr, beta1, beta2, eps,
                                              c1, c2);
  return hip_status(h, hipGetLastError(), "adam");
}

const char* fno_last_error(fno_handle h) { return h ? h->err.c_str() : "null handle"; }

void fno_destroy(fno_handle h) {
  if (!h) return;
  if (h->st) (void)hipStreamSynchronize(h->st);
  for (void* ptr : h->allocs) (void)hipFree(ptr);
  if (h->own_stream) (void)hipStreamDestroy(h->st);
  delete h;
}

}  // extern "C"
