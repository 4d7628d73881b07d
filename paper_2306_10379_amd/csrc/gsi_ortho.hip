// Standalone orthonormalization of a tall block by two passes of Cholesky QR: X <- X R^{-1}
// with R^T R = X^T X, twice. It is the re-orthonormalization step of the iteration (the
// start block, a warm start, a precision switch) offered on a caller's block, row-major with
// leading dimension p (no padding), float64, in place.
//
// k_ortho_gram forms per-workgroup partial sums of the upper blocks of X^T X, k_ortho_sum adds
// them in a fixed order (the result repeats bit for bit), k_ortho_chol factors the sum and
// inverts the factor, and k_ortho_apply multiplies X by R^{-1}; the first pass's k_ortho_apply
// also forms the partial sums of the second pass's Gram from the rows it writes, which are in
// its registers. A failed factorization (a non-positive or tiny pivot: X is rank deficient or
// not finite) sets a flag that makes the later kernels of the call return without touching X.
//
// The block is read three times and written twice, which bounds the call at large n: with the
// products on MFMA the kernels take 270 us at n = 1,000,003, p = 30 (1.2 GB at 4.4 TB/s), where
// they took 4020 us with element-wise products out of LDS (950 us a Gram, 860 us an apply).
//
// Scratch (per call): the partial sums, R^{-1} and two flags. gsi_orthonormalize allocates
// it for the call; gsi_orthonormalize_noalloc uses a file-scope device array instead, so
// that callers that cannot allocate device memory can call it.
#include <hip/hip_runtime.h>

#include <mutex>
#include <stdint.h>

#include "../../include/gsi.h"
#include "gsi_dense_dev.h"

namespace {

using gsi::d4;
using gsi::mfma;

constexpr int OWG = 512;        // threads per workgroup of the tall passes: one workgroup per CU
constexpr int OMAXP = 64;       // largest block width
constexpr int OMAXWG = 256;     // workgroups of the Gram pass (the partial sums they write)
constexpr int OMAXP2 = OMAXP * (OMAXP + 1) / 2;
// scratch layout in doubles: partials [OMAXWG * OMAXP2], R^{-1} [OMAXP * OMAXP], flags
constexpr size_t OFF_RINV = (size_t)OMAXWG * OMAXP2;
constexpr size_t OFF_FLAGS = OFF_RINV + (size_t)OMAXP * OMAXP;
constexpr size_t SCRATCH_DOUBLES = OFF_FLAGS + 64;

// Scratch of gsi_orthonormalize_noalloc: 4.3 MB on every device the library runs on, held
// until the process ends. Host code must not pass this name to a kernel (it is a host-side
// stand-in there): it uses the device address from hipGetSymbolAddress.
__device__ __align__(256) double scratch[SCRATCH_DOUBLES];

// Orders the LDS accesses of a wave's lanes among each other.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Upper 16 x 16 blocks (ib <= jb) of a Gram of NB column blocks.
template <int NB>
constexpr int UB = NB * (NB + 1) / 2;

// acc += Y^T Y for 16 rows of Y in the MFMA layout y[cb][s]: lane (g, c) holds row 4 s + g,
// column 16 cb + c, which is both operands' layout.
template <int NB>
__device__ __forceinline__ void gram16(const double (&y)[NB][4], d4 (&acc)[UB<NB>]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    int k = 0;
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int jb = ib; jb < NB; ++jb, ++k) acc[k] = mfma(y[ib][s], y[jb][s], acc[k]);
  }
}

// Sums the waves' blocks in wave order through LDS and writes the workgroup's partial sums,
// entry (i, j), i <= j, at its place in row-major order of the upper triangle.
template <int NB>
__device__ __forceinline__ void store_gram(int p, const d4 (&acc)[UB<NB>], double* lds, double* __restrict__ partials) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  for (int k = 0; k < OWG / 64; ++k) {
    __syncthreads();
    if (w == k)
#pragma unroll
      for (int b = 0; b < UB<NB>; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double* at = lds + (b * 4 + r) * 64 + l;
          *at = k ? *at + acc[b][r] : acc[b][r];
        }
  }
  __syncthreads();
  double* out = partials + (int64_t)blockIdx.x * (p * (p + 1) / 2);
  for (int t = w; t < UB<NB> * 4; t += OWG / 64) {
    int ib = 0, b = t >> 2;
    while (b >= NB - ib) b -= NB - ib++;
    const int i = 16 * ib + g + 4 * (t & 3), j = 16 * (ib + b) + c;
    if (i <= j && j < p) out[i * p - i * (i - 1) / 2 + j - i] = lds[t * 64 + l];
  }
}

// Partial sums of X^T X, 16-row tiles dealt to the waves of the grid; U tiles' loads (8 bytes a
// lane: rows of p doubles have no wider alignment) are in flight together, which is what the
// pass needs to run at the read rate.
template <int NB>
__global__ __launch_bounds__(OWG, 2) void k_ortho_gram(int64_t n, int p, const double* __restrict__ X,
                                                       double* __restrict__ partials) {
  constexpr int U = NB == 1 ? 8 : (NB == 2 ? 4 : 2);
  __shared__ double lds[UB<NB> * 256];
  const int l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  d4 acc[UB<NB>];
#pragma unroll
  for (int b = 0; b < UB<NB>; ++b) acc[b] = d4{0.0, 0.0, 0.0, 0.0};
  const int64_t nt = (n + 15) / 16, stride = (int64_t)gridDim.x * (OWG / 64);
  for (int64_t t = (int64_t)blockIdx.x * (OWG / 64) + (threadIdx.x >> 6); t < nt; t += U * stride) {
    double y[U][NB][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int64_t row = (t + u * stride) * 16 + 4 * s + g;
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          const bool ok = row < n && 16 * cb + c < p;
          y[u][cb][s] = ok ? X[row * p + 16 * cb + c] : 0.0;
        }
      }
#pragma unroll
    for (int u = 0; u < U; ++u) gram16<NB>(y[u], acc);
  }
  store_gram<NB>(p, acc, lds, partials);
}

// G = sum of the nb partials, 64 values and SLICES slices of the partials to a workgroup, added
// in a fixed order (one workgroup adding all of them took 80 us; 4 slices, 64 dependent loads
// each, 20 us).
constexpr int SLICES = 16;
__global__ __launch_bounds__(64 * SLICES) void k_ortho_sum(int np, int nb, const double* __restrict__ partials,
                                                           double* __restrict__ G, const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ double part[SLICES][64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6, e = blockIdx.x * 64 + l;
  double s = 0.0;
  if (e < np)
#pragma unroll 4
    for (int b = w; b < nb; b += SLICES) s += partials[(int64_t)b * np + e];
  part[w][l] = s;
  __syncthreads();
  if (w == 0 && e < np) {
    for (int k = 1; k < SLICES; ++k) s += part[k][l];
    G[e] = s;
  }
}

// One workgroup: G = L L^T (G: the upper triangle by rows), rinv = L^{-T} (upper triangular, 64
// x 64 row-major, zero elsewhere); G and rinv may overlap. flag_out = 1 when a pivot is not
// above 1e-13 max_i G_ii (or not finite), or when flag_in (nullable) is already set.
__global__ __launch_bounds__(256) void k_ortho_chol(int p, const double* G, double* rinv,
                                                    const int* __restrict__ flag_in, int* __restrict__ flag_out) {
  constexpr int LD = gsi::DLD<OMAXP>;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double* A = reinterpret_cast<double*>(lds_raw);
  double* M = A + OMAXP * LD;
  if (flag_in && *flag_in) {
    if (threadIdx.x == 0) *flag_out = 1;
    return;
  }
  const int m = 16 * ((p + 15) / 16), l = threadIdx.x & 63;
  for (int i = threadIdx.x >> 6; i < m; i += 4)
    if (l < m) {
      const int a = i < l ? i : l, b = i < l ? l : i;
      A[i * LD + l] = b < p ? G[a * p - a * (a - 1) / 2 + b - a] : 0.0;
    }
  __syncthreads();
  double dmax = l < p ? A[l * LD + l] : 0.0;
  dmax = gsi::wave_max(dmax);
  const bool bad = gsi::chol_lds<OMAXP, false>(p, A, 1e-13 * dmax);
  gsi::inv_chol<OMAXP>(p, A, M, LD);
  for (int i = threadIdx.x >> 6; i < OMAXP; i += 4) rinv[i * OMAXP + l] = i < p && l < p ? M[i * LD + l] : 0.0;
  if (threadIdx.x == 0) *flag_out = bad ? 1 : 0;
}

// X <- X R^{-1} in place; GRAM: also the partial sums of the result's Gram. Returns at once
// when the factorization failed. A wave takes U tiles of 16 rows at a time: they are contiguous
// in memory, are read element by element in order (the next U while these multiply) and staged
// in the wave's own LDS rows, 16 NB + 2 apart so that the reads of the product's left operand
// are free of bank conflicts; the blocks of R^{-1} on and above the diagonal stay in registers
// (in LDS where the Gram's blocks leave no room: 4 column blocks).
template <int NB, bool GRAM>
__global__ __launch_bounds__(OWG, 2) void k_ortho_apply(int64_t n, int p, double* __restrict__ X,
                                                        const double* __restrict__ rinv, const int* __restrict__ flag,
                                                        double* __restrict__ partials) {
  if (*flag) return;
  constexpr int U = NB == 1 ? 4 : (NB == 2 ? 2 : 1), PS = 16 * NB + 2, NW = OWG / 64;
  constexpr int STAGE = NW * U * 16 * PS, GR = GRAM ? UB<NB> * 256 : 0;
  constexpr bool R_LDS = NB == 4 && GRAM;
  constexpr int RS = OMAXP + 16;  // row stride of R^{-1} in LDS: 4 rows a load, on all banks
  __shared__ double sr[R_LDS ? OMAXP * RS : 1];
  __shared__ double lds[STAGE > GR ? STAGE : GR];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
  double* mine = lds + w * U * 16 * PS;
  double rb[R_LDS ? 1 : UB<NB>][4];  // block (kb, jb), kb <= jb: lane (g, c) holds row 16 kb + 4 s + g, column 16 jb + c
  if constexpr (R_LDS) {
    for (int e = threadIdx.x; e < OMAXP * OMAXP; e += OWG) sr[(e >> 6) * RS + (e & 63)] = rinv[e];
    __syncthreads();
  } else {
    int k = 0;
#pragma unroll
    for (int kb = 0; kb < NB; ++kb)
#pragma unroll
      for (int jb = kb; jb < NB; ++jb, ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) rb[k][s] = rinv[(16 * kb + 4 * s + g) * OMAXP + 16 * jb + c];
  }
  d4 acc[GRAM ? UB<NB> : 1];
  if constexpr (GRAM)
#pragma unroll
    for (int b = 0; b < UB<NB>; ++b) acc[b] = d4{0.0, 0.0, 0.0, 0.0};
  // element e = l + 64 i of the U tiles is (row e / p, column e mod p): e < 1024 and p <= 64, so
  // e / p = e ceil(2^16 / p) / 2^16
  const uint32_t magic = (65536u + p - 1) / p;
  const int count = U * 16 * p;
  constexpr int NI = U * 4 * NB;  // loads per lane
  for (int e = l; e < U * 16 * PS; e += 64) mine[e] = 0.0;  // columns p .. 16 NB stay zero
  const int64_t total = n * p, stride = (int64_t)gridDim.x * NW;
  const int64_t ng = (n + U * 16 - 1) / (U * 16);
  int64_t t = (int64_t)blockIdx.x * NW + w;
  double in[NI];
  auto load = [&](int64_t tt) {
    const int64_t base = tt * count;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = l + 64 * i;
      in[i] = tt < ng && e < count && base + e < total ? X[base + e] : 0.0;
    }
  };
  load(t);
  for (; t < ng; t += stride) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = l + 64 * i;
      const int row = (int)((uint32_t)e * magic >> 16);
      if (e < count) mine[row * PS + e - row * p] = in[i];
    }
    load(t + stride);
    wave_order();  // the wave's LDS rows are its own: its reads only follow its own writes
#pragma unroll
    for (int u = 0; u < U; ++u) {
      d4 y[NB];
#pragma unroll
      for (int jb = 0; jb < NB; ++jb) y[jb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        int k = 0;
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
          const double a = mine[(16 * u + c) * PS + 16 * kb + 4 * s + g];
#pragma unroll
          for (int jb = kb; jb < NB; ++jb, ++k) {
            double b;
            if constexpr (R_LDS) b = sr[(16 * kb + 4 * s + g) * RS + 16 * jb + c];
            else b = rb[k][s];
            y[jb] = mfma(a, b, y[jb]);
          }
        }
      }
      const int64_t r0 = (t * U + u) * 16 + g;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r0 + 4 * r < n)
#pragma unroll
          for (int jb = 0; jb < NB; ++jb)
            if (16 * jb + c < p) X[(r0 + 4 * r) * p + 16 * jb + c] = y[jb][r];
      if constexpr (GRAM) {
        double yy[NB][4];  // rows g + 4 r of the product are the Gram's rows 4 s + g (rows past n are zero)
#pragma unroll
        for (int jb = 0; jb < NB; ++jb)
#pragma unroll
          for (int r = 0; r < 4; ++r) yy[jb][r] = y[jb][r];
        gram16<NB>(yy, acc);
      }
    }
    wave_order();
  }
  if constexpr (GRAM) store_gram<NB>(p, acc, lds, partials);
}

// The two passes on the stream; scratch is a device pointer of SCRATCH_DOUBLES doubles.
// Returns the flag of the second pass (read back after a synchronization).
template <int NB>
gsi_status run_cholqr2(int64_t n, int p, double* X, double* scr, hipStream_t st) {
  constexpr int CHOL_LDS = 2 * OMAXP * gsi::DLD<OMAXP> * (int)sizeof(double);
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(k_ortho_chol), hipFuncAttributeMaxDynamicSharedMemorySize,
                          CHOL_LDS) != hipSuccess)
    return GSI_EDEVICE;
  const int64_t t = (n + 127) / 128;  // a 16-row tile for each of the 8 waves
  const int nb = (int)(t < OMAXWG ? t : OMAXWG), np = p * (p + 1) / 2;
  double* partials = scr;
  double* rinv = scr + OFF_RINV;
  int* flags = reinterpret_cast<int*>(scr + OFF_FLAGS);
  k_ortho_gram<NB><<<nb, OWG, 0, st>>>(n, p, X, partials);
  k_ortho_sum<<<(np + 63) / 64, 64 * SLICES, 0, st>>>(np, nb, partials, rinv, nullptr);
  k_ortho_chol<<<1, 256, CHOL_LDS, st>>>(p, rinv, rinv, nullptr, flags);
  k_ortho_apply<NB, true><<<nb, OWG, 0, st>>>(n, p, X, rinv, flags, partials);
  k_ortho_sum<<<(np + 63) / 64, 64 * SLICES, 0, st>>>(np, nb, partials, rinv, flags);
  k_ortho_chol<<<1, 256, CHOL_LDS, st>>>(p, rinv, rinv, flags, flags + 1);
  k_ortho_apply<NB, false><<<nb, OWG, 0, st>>>(n, p, X, rinv, flags + 1, nullptr);
  if (hipGetLastError() != hipSuccess) return GSI_EDEVICE;
  int flag = 0;
  if (hipMemcpyAsync(&flag, flags + 1, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess) return GSI_EDEVICE;
  if (hipStreamSynchronize(st) != hipSuccess) return GSI_EDEVICE;
  return flag ? GSI_BREAKDOWN : GSI_OK;
}

gsi_status run(int64_t n, int p, double* X, double* scr, hipStream_t st) {
  if (p <= 16) return run_cholqr2<1>(n, p, X, scr, st);
  if (p <= 32) return run_cholqr2<2>(n, p, X, scr, st);
  if (p <= 48) return run_cholqr2<3>(n, p, X, scr, st);
  return run_cholqr2<4>(n, p, X, scr, st);
}

gsi_status check_args(const double* X, int64_t n, int32_t p) {
  if (!X || p < 1 || n < p) return GSI_EINVAL;
  if (p > OMAXP) return GSI_EUNSUPPORTED;
  return GSI_OK;
}

// Device address of `scratch` on each device, looked up once per device with that device
// current (each device holds its own copy of the array at its own address).
constexpr int MAXDEV = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[MAXDEV] = {nullptr};

gsi_status scratch_for_current_device(double** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAXDEV) return GSI_EDEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return GSI_EDEVICE;
    g_scratch_ptr[dev] = reinterpret_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return GSI_OK;
}

}  // namespace

extern "C" {

gsi_status gsi_orthonormalize(double* X, int64_t n, int32_t p, void* hip_stream) {
  gsi_status s = check_args(X, n, p);
  if (s != GSI_OK) return s;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  void* scr = nullptr;
  if (hipMalloc(&scr, SCRATCH_DOUBLES * sizeof(double)) != hipSuccess) return GSI_ENOMEM;
  s = run(n, p, X, reinterpret_cast<double*>(scr), st);
  if (s == GSI_EDEVICE) (void)hipStreamSynchronize(st);
  (void)hipFree(scr);
  return s;
}

gsi_status gsi_orthonormalize_noalloc(double* X, int64_t n, int32_t p, void* hip_stream) {
  gsi_status s = check_args(X, n, p);
  if (s != GSI_OK) return s;
  double* scr = nullptr;
  s = scratch_for_current_device(&scr);
  if (s != GSI_OK) return s;
  return run(n, p, X, scr, reinterpret_cast<hipStream_t>(hip_stream));
}

}  // extern "C"
