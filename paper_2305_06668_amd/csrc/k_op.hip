// Operator application Y = A W for the matrix kinds the solver accepts
// (Alg. 1: the products A X^[0] and A W^[k]; the method is matrix-free,
// Sec. 3.1, so the operator is an input, not part of the method).
//
//   * CSR SpMM: in k_spmm.hip.
//   * dense: HBM-bound on A, which is read once for up to 16 columns.
#include "internal.h"

namespace lobpcg {

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ---------------------------------------------------------------------------
// dense: Y (n x ncols) = A (n x n, lda) W (n x ncols), up to 16 columns per
// launch, on the MFMA 16x16x4.
//
// A workgroup owns RT tiles of 16 rows; its NW waves take chunks of 32 columns
// of A in turn and add up their tiles through LDS at the end, in a fixed order.
// A chunk's products go to NA accumulators, which are added in a tree and then
// to the wave's sums: no chain of additions is longer than with the sums over
// the lanes of a wave per row that this kernel replaced (n / 64 terms and six
// levels), and the error is no larger (n = 2000, 5999, 20000 fp64, relative:
// 2.0e-16, 2.8e-16, 4.5e-16 where it was 2.2e-16, 3.5e-16, 6.1e-16; with one
// accumulator throughout 3.9e-16 at n = 2000).
// A load takes 16 bytes per lane: row lane % 16, VE adjacent columns for each
// of the four k of an MFMA (lane / 16), 64 bytes of a row; the W operand of
// lane (g, c) is W[k][c] of the same k, columns past ncols being copies of the
// last one that are not stored.  The next chunk is loaded while the current
// one is multiplied.  Loads need element alignment only.
// SPREAD: workgroup b begins 37 b strides of the workgroup further along its
// rows (and wraps at their end), so that the workgroups, which run in step, do
// not all read the same columns at a time: rows of 64 KB lie on the same
// memory channels then.  A sum's additions are as many, in another order.
// What bounds it: the read of A, once for up to 16 columns (n = 2e4 fp64: 630
// us = 5.1 TB/s, where a plain sum reads 6.0; 8 columns at a time by scalar
// products, eight rows per wave: 664 us for 8, 1330 for 16); at small n the
// latency of a wave's few chunks (n = 2000, 13 columns: 15 us; 65 before, as
// 63 workgroups and a packing pass for each 8 columns).  Chunks of 64 columns,
// a contiguous range per wave and the non-temporal hint were all slower (the
// hint 790 against 656 us, and A of up to 256 MB is read again from the
// memory-side cache).
typedef double __attribute__((ext_vector_type(2), aligned(8))) v2d_u;
typedef float __attribute__((ext_vector_type(4), aligned(4))) v4f_u;
template <typename T> struct DenseTypes;
template <> struct DenseTypes<double> { typedef d4 Acc; typedef v2d_u Vec; };
template <> struct DenseTypes<float> { typedef f4 Acc; typedef v4f_u Vec; };
__device__ __forceinline__ d4 dmma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 dmma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// v[0] + ... by halves (N a power of two)
template <typename T, int N>
__device__ __forceinline__ T tree_sum(T (&v)[N]) {
#pragma unroll
  for (int h = N / 2; h >= 1; h /= 2)
#pragma unroll
    for (int q = 0; q < h; ++q) v[q] += v[q + h];
  return v[0];
}

template <typename T, int RT, int NW, int NA, bool SPREAD>
__global__ __launch_bounds__(64 * NW) void k_dense_mfma(const T* __restrict__ A, int64_t lda,
                                                        const T* __restrict__ W, int64_t ldw,
                                                        T* __restrict__ Y, int64_t ldy, int ncols,
                                                        int64_t n) {
  typedef typename DenseTypes<T>::Acc Acc;
  typedef typename DenseTypes<T>::Vec Vec;
  constexpr int VE = 16 / (int)sizeof(T);  // columns of A per load and lane
  constexpr int KC = 32;                   // columns of A per chunk
  constexpr int NI = KC / (4 * VE);        // loads per row tile and chunk
  __shared__ T part[NW][RT * 16][17];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int64_t r0 = (int64_t)blockIdx.x * (16 * RT);
  const T* ap[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) ap[t] = A + min(r0 + 16 * t + r, n - 1) * lda + VE * g;
  const T* wp = W + min(r, ncols - 1) + (int64_t)(VE * g) * ldw;
  Acc sum[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[t][e] = T(0);
  struct Chunk {
    Vec a[RT][NI];
    T w[NI][VE];
  };
  const int64_t nfull = n & ~(int64_t)(KC - 1);
  constexpr int64_t step = KC * NW;
  const int64_t first = SPREAD ? (int64_t)(blockIdx.x * 37 % (uint32_t)(nfull / step)) * step : 0;
  auto load = [&](Chunk& c, int64_t k0) {
    if (SPREAD) {
      k0 += first;
      if (k0 >= nfull) k0 -= nfull;
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int i = 0; i < NI; ++i) c.a[t][i] = *reinterpret_cast<const Vec*>(ap[t] + k0 + 4 * VE * i);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < VE; ++e) c.w[i][e] = wp[(k0 + 4 * VE * i + e) * ldw];
  };
  auto mul = [&](const Chunk& c) {
    Acc acc[NA][RT];
#pragma unroll
    for (int q = 0; q < NI * VE; ++q)
#pragma unroll
      for (int t = 0; t < RT; ++t)
        acc[q % NA][t] = dmma(c.a[t][q / VE][q % VE], c.w[q / VE][q % VE], q < NA ? Acc{} : acc[q % NA][t]);
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        T v[NA];
#pragma unroll
        for (int q = 0; q < NA; ++q) v[q] = acc[q][t][e];
        sum[t][e] += tree_sum(v);
      }
  };
  int64_t k = KC * wave;
  Chunk c0, c1;
  if (k < nfull) load(c0, k);
  while (k < nfull) {
    if (k + step < nfull) load(c1, k + step);
    mul(c0);
    k += step;
    if (k >= nfull) break;
    if (k + step < nfull) load(c0, k + step);
    mul(c1);
    k += step;
  }
  if (k == nfull && nfull < n) {  // the wave whose chunk is the last, partial one
    Chunk c;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < VE; ++e) {
        const int64_t kk = nfull + 4 * VE * i + e;
        const bool in = kk + VE * g < n;
        c.w[i][e] = in ? wp[kk * ldw] : T(0);
#pragma unroll
        for (int t = 0; t < RT; ++t) c.a[t][i][e] = in ? ap[t][kk] : T(0);
      }
    mul(c);
  }
  // accumulator register e of lane (g, c): row 4 e + g (fp64), 4 g + e (fp32)
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave][16 * t + (sizeof(T) == 8 ? 4 * e + g : 4 * g + e)][r] = sum[t][e];
  __syncthreads();
  for (int q = threadIdx.x; q < RT * 256; q += 64 * NW) {
    const int i = q >> 4, j = q & 15;
    T v[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) v[w] = part[w][i][j];
    const T y = tree_sum(v);
    if (r0 + i < n && j < ncols) Y[(r0 + i) * ldy + j] = y;
  }
}

// At most MC columns by scalar products: a wave owns R rows, lanes stride their
// columns, and the sums are reduced across the wave at the end.
template <typename T, int R, int MC>
__global__ __launch_bounds__(256) void k_dense(const T* __restrict__ A, int64_t lda,
                                               const T* __restrict__ W, int64_t ldw,
                                               T* __restrict__ Y, int64_t ldy, int ncols,
                                               int64_t n) {
  const int lane = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t r0 = gw * R;
  if (r0 >= n) return;
  T acc[R][MC];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < MC; ++j) acc[r][j] = T(0);
  const T* arow[R];
#pragma unroll
  for (int r = 0; r < R; ++r) arow[r] = A + min(r0 + r, n - 1) * lda;
  for (int64_t c = lane; c < n; c += 64) {
    T w[MC];
#pragma unroll
    for (int j = 0; j < MC; ++j) w[j] = (j < ncols) ? W[c * ldw + j] : T(0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T a = arow[r][c];
#pragma unroll
      for (int j = 0; j < MC; ++j) acc[r][j] += a * w[j];
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      T v = acc[r][j];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
      acc[r][j] = v;
    }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r0 + r < n)
#pragma unroll
        for (int j = 0; j < MC; ++j)
          if (j < ncols) Y[(r0 + r) * ldy + j] = acc[r][j];
  }
}

// Two or four fp64 columns of a compact block (W rows of 16 bytes, aligned as
// A's are): a wave owns eight rows, a lane two adjacent columns of A per step,
// so that a W row fetched serves eight rows of A.  A is read with the
// non-temporal hint: past the 256 MB of the memory-side cache a part of it is
// then found there by the next product (n = 8192, 4 columns: 86 us, 117
// without; 10000: 196, 215).
template <int MC>
__global__ __launch_bounds__(256) void k_dense_vec(const double* __restrict__ A, int64_t lda,
                                                   const double* __restrict__ W, int64_t ldw,
                                                   double* __restrict__ Y, int64_t ldy, int64_t n) {
  constexpr int R = 8;
  typedef double __attribute__((ext_vector_type(2))) V;
  const int lane = threadIdx.x & 63;
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
  if (r0 >= n) return;
  double acc[R][MC];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < MC; ++j) acc[r][j] = 0.0;
  const double* arow[R];
#pragma unroll
  for (int r = 0; r < R; ++r) arow[r] = A + min(r0 + r, n - 1) * lda;
  const int64_t nfull = n & ~(int64_t)127;
#pragma unroll 1
  for (int64_t c = 2 * lane; c < nfull; c += 128) {
    V a[R], w[2][MC / 2];
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = __builtin_nontemporal_load(reinterpret_cast<const V*>(arow[r] + c));
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int q = 0; q < MC / 2; ++q) w[e][q] = *reinterpret_cast<const V*>(W + (c + e) * ldw + 2 * q);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int j = 0; j < MC; ++j) acc[r][j] += a[r][e] * w[e][j / 2][j % 2];
  }
  for (int64_t c = nfull + lane; c < n; c += 64) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double a = arow[r][c];
#pragma unroll
      for (int j = 0; j < MC; ++j) acc[r][j] += a * W[c * ldw + j];
    }
  }
  double mine = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      double v = acc[r][j];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
      if (lane == r * MC + j) mine = v;
    }
  const int r = lane / MC, j = lane % MC;
  if (r < R && r0 + r < n) Y[(r0 + r) * ldy + j] = mine;
}

template <typename T, int R, int MC>
static void dense_scalar(const T* A, int64_t lda, const T* W, int64_t ldw, T* Y, int64_t ldy, int nc, int64_t n,
                         hipStream_t s) {
  hipLaunchKernelGGL((k_dense<T, R, MC>), dim3(cdiv(cdiv(n, R), 4)), dim3(256), 0, s, A, lda, W, ldw, Y, ldy, nc, n);
}

// Up to four fp64 columns whose rows lie close together (ldw <= 4): the MFMA
// kernel multiplies 16 columns whatever their number, and its workgroups of 32
// rows are more than one but fewer than two to a CU between n = 8192 and
// 16384.  False: no launch, the MFMA kernel is the faster one.  us at n, as
// launched here and by the MFMA kernel:
//   1 column    1500: 8.2, 11.0   5000: 35, 52   9000: 126, 185   12000: 192, 259   20000: 547, 622
//   2 columns   1500: 8.2, 11.2   5000: 48, 52   9000: 146, 185   12000: 200, 259   20000: 518, 623
//   3 columns   1500: 8.1, 11.1   5000: 40, 52   9000: 156, 186   14000: 287, 305   (7000: 89, 81)
//   4 columns   1500: 8.8, 11.1   5000: 47, 52   9000: 180, 186   16000: 344, 360   8192: 86, 117
static bool dense_few(const double* A, int64_t lda, const double* W, int64_t ldw, double* Y, int64_t ldy, int nc,
                      int64_t n, hipStream_t s) {
  if (n < 1800) {  // two rows to a wave: enough waves
    if (nc == 1) dense_scalar<double, 2, 1>(A, lda, W, ldw, Y, ldy, nc, n, s);
    else if (nc == 2) dense_scalar<double, 2, 2>(A, lda, W, ldw, Y, ldy, nc, n, s);
    else if (nc == 3) dense_scalar<double, 2, 3>(A, lda, W, ldw, Y, ldy, nc, n, s);
    else dense_scalar<double, 2, 4>(A, lda, W, ldw, Y, ldy, nc, n, s);
    return true;
  }
  if (n < 16 * 256) return false;
  const bool vec = lda % 2 == 0 && ldw % 2 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(W) % 16 == 0;
  const int grid8 = cdiv(cdiv(n, 8), 4);
  if (vec && nc == 4)
    hipLaunchKernelGGL(k_dense_vec<4>, dim3(grid8), dim3(256), 0, s, A, lda, W, ldw, Y, ldy, n);
  else if (vec && nc == 2)
    hipLaunchKernelGGL(k_dense_vec<2>, dim3(grid8), dim3(256), 0, s, A, lda, W, ldw, Y, ldy, n);
  else if (nc == 1 && n < 12500)
    dense_scalar<double, 4, 1>(A, lda, W, ldw, Y, ldy, nc, n, s);
  else if (nc == 1)  // (fewer waves in flight keep more of W in L2: 1 column by <4, 1> at 20000 602 us)
    dense_scalar<double, 4, 4>(A, lda, W, ldw, Y, ldy, nc, n, s);
  else if (nc == 2 && n < 12500)
    dense_scalar<double, 4, 2>(A, lda, W, ldw, Y, ldy, nc, n, s);
  else if (nc == 3 && (n < 5800 || (n > 8192 && n < 12500)))
    dense_scalar<double, 4, 3>(A, lda, W, ldw, Y, ldy, nc, n, s);
  else if (nc == 3 && n >= 12500 && n <= 16384)
    dense_scalar<double, 8, 3>(A, lda, W, ldw, Y, ldy, nc, n, s);
  else
    return false;
  return true;
}
static bool dense_few(const float*, int64_t, const float*, int64_t, float*, int64_t, int, int64_t, hipStream_t) {
  return false;  // (1500: 8.7 us by the MFMA kernel and 8.1 by scalar products, 12000: 108 and 125)
}

template <typename T>
static hipError_t dense_any(const T* A, int64_t lda, const T* W, int64_t ldw, T* Y, int64_t ldy,
                            int ncols, int64_t n, hipStream_t s) {
  if (n < 1 || ncols < 1) return hipErrorInvalidValue;
  // Below one tile per CU a workgroup is 8 waves (n = 3000 fp32: 10.7 us, 12.0
  // with 4; n = 4000 fp64: 26.9 and 24.4).  From 6000 rows two tiles share the
  // loads of W in fp64 (n = 6007: 69 us, 75 with one; 4000: 41 and 24).  Rows
  // of doubles that are not all aligned to 16 bytes cost the MFMA kernel's
  // loads half again their time: up to 4 columns the scalar products, which
  // load 8 bytes per lane, are faster then (n = 9001, 1 column: 135 against
  // 199 us, 4: 177 and 200, 8: 316 and 203; n = 777, 1 column: 9.4 and 8.9).
  const bool odd = sizeof(T) == 8 && (lda % 2 != 0 || reinterpret_cast<uintptr_t>(A) % 16 != 0);
  // Workgroups apart: fp64 6016 rows, 16 columns 65 us, 67 in step; 8192: 98 and
  // 108, compact 8 columns 96 and 114; 16320: 371 and 411; 20000: 657 and 644.
  // fp32, 9000: 107 and 97; 14000: 174 and 203; 16320, 8 of 24 columns: 211 and
  // 287; 20000, compact 8 columns: 320 and 315.
  const bool spread = n >= (sizeof(T) == 8 ? 6000 : 13000) && n < 17000;
  for (int c0 = 0; c0 < ncols; c0 += 16) {
    const int nc = std::min(16, ncols - c0);
    if (nc <= 4 && ldw <= 4 && dense_few(A, lda, W + c0, ldw, Y + c0, ldy, nc, n, s))
      ;
    else if (odd && nc <= 4 && n >= 16 * 256)
      hipLaunchKernelGGL((k_dense<T, 4, 4>), dim3(cdiv(cdiv(n, 4), 4)), dim3(256), 0, s, A, lda, W + c0, ldw, Y + c0,
                         ldy, nc, n);
    else if (n < 16 * 256)
      hipLaunchKernelGGL((k_dense_mfma<T, 1, 8, 8, false>), dim3(cdiv(n, 16)), dim3(512), 0, s, A, lda, W + c0, ldw, Y + c0,
                         ldy, nc, n);
    else if (sizeof(T) == 8 && spread)
      hipLaunchKernelGGL((k_dense_mfma<T, 2, 4, 2, true>), dim3(cdiv(n, 32)), dim3(256), 0, s, A, lda, W + c0, ldw,
                         Y + c0, ldy, nc, n);
    else if (sizeof(T) == 8 && n >= 6000)
      hipLaunchKernelGGL((k_dense_mfma<T, 2, 4, 2, false>), dim3(cdiv(n, 32)), dim3(256), 0, s, A, lda, W + c0, ldw,
                         Y + c0, ldy, nc, n);
    else if (spread)
      hipLaunchKernelGGL((k_dense_mfma<T, 1, 4, 4, true>), dim3(cdiv(n, 16)), dim3(256), 0, s, A, lda, W + c0, ldw,
                         Y + c0, ldy, nc, n);
    else
      hipLaunchKernelGGL((k_dense_mfma<T, 1, 4, 4, false>), dim3(cdiv(n, 16)), dim3(256), 0, s, A, lda, W + c0, ldw,
                         Y + c0, ldy, nc, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t dense_apply_f64(const double* A, int64_t lda, const double* W, int64_t ldw, double* Y,
                           int64_t ldy, int ncols, int64_t n, hipStream_t s) {
  return dense_any<double>(A, lda, W, ldw, Y, ldy, ncols, n, s);
}
hipError_t dense_apply_f32(const float* A, int64_t lda, const float* W, int64_t ldw, float* Y,
                           int64_t ldy, int ncols, int64_t n, hipStream_t s) {
  return dense_any<float>(A, lda, W, ldw, Y, ldy, ncols, n, s);
}

// ---------------------------------------------------------------------------
// CSR structure check (run once when the operator is set): row pointers
// non-decreasing from 0 to nnz, every column index inside [0, n).

__global__ void k_csr_check(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                            int64_t n, int64_t nnz, int* __restrict__ bad) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0 && (rp[0] != 0 || (int64_t)rp[n] != nnz)) atomicOr(bad, 1);
  if (i >= n) return;
  const int32_t e0 = rp[i], e1 = rp[i + 1];
  if (e1 < e0 || e0 < 0 || (int64_t)e1 > nnz) {
    atomicOr(bad, 2);
    return;
  }
  for (int32_t e = e0; e < e1; ++e) {
    const int32_t c = ci[e];
    if (c < 0 || (int64_t)c >= n) {
      atomicOr(bad, 4);
      return;
    }
  }
}
hipError_t csr_check(const int32_t* rp, const int32_t* ci, int64_t n, int64_t nnz, int* bad,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_csr_check, dim3(cdiv(n, 256)), dim3(256), 0, s, rp, ci, n, nnz, bad);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gershgorin bound max_i sum_j |a_ij| (used by the precision switch)

__device__ __forceinline__ double block_max(double v, double* sh) {
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
  for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = fmax(r, sh[i]);
  return r;
}

__global__ __launch_bounds__(256) void k_csr_rowabs(const int32_t* __restrict__ rp,
                                                    const double* __restrict__ val, int64_t n,
                                                    double* __restrict__ part) {
  __shared__ double sh[4];
  double best = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    double s = 0.0;
    for (int e = rp[i]; e < rp[i + 1]; ++e) s += fabs(val[e]);
    best = fmax(best, s);
  }
  best = block_max(best, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = best;
}

__global__ __launch_bounds__(256) void k_dense_rowabs(const double* __restrict__ A, int64_t lda,
                                                      int64_t n, double* __restrict__ part) {
  __shared__ double sh[4];
  double best = 0.0;
  // one wave per row
  const int lane = threadIdx.x & 63;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {
    double s = 0.0;
    for (int64_t j = lane; j < n; j += 64) s += fabs(A[i * lda + j]);
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    best = fmax(best, s);
  }
  best = block_max(best, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = best;
}

__global__ void k_max_final(const double* __restrict__ part, int nblk, double* __restrict__ out) {
  __shared__ double sh[4];
  double best = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) best = fmax(best, part[i]);
  best = block_max(best, sh);
  if (threadIdx.x == 0) *out = best;
}

hipError_t csr_norm_bound(const int32_t* rp, const double* val, int64_t n, double* part,
                          double* out, hipStream_t s) {
  const int grid = (int)std::min<int64_t>(kStreamBlocks, cdiv(n, 256));
  hipLaunchKernelGGL(k_csr_rowabs, dim3(grid), dim3(256), 0, s, rp, val, n, part);
  hipLaunchKernelGGL(k_max_final, dim3(1), dim3(256), 0, s, part, grid, out);
  return hipGetLastError();
}

hipError_t dense_norm_bound(const double* A, int64_t lda, int64_t n, double* part, double* out,
                            hipStream_t s) {
  const int grid = (int)std::min<int64_t>(kStreamBlocks, cdiv(n, 4));
  hipLaunchKernelGGL(k_dense_rowabs, dim3(grid), dim3(256), 0, s, A, lda, n, part);
  hipLaunchKernelGGL(k_max_final, dim3(1), dim3(256), 0, s, part, grid, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// diagonals (inputs of the Jacobi preconditioner)

__global__ void k_csr_diag(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                           const double* __restrict__ val, int64_t n, double* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  double v = 0.0;
  for (int e = rp[i]; e < rp[i + 1]; ++e)
    if (ci[e] == i) v += val[e];
  d[i] = v;
}
hipError_t csr_diag(const int32_t* rp, const int32_t* ci, const double* val, int64_t n,
                    double* diag, hipStream_t s) {
  hipLaunchKernelGGL(k_csr_diag, dim3(cdiv(n, 256)), dim3(256), 0, s, rp, ci, val, n, diag);
  return hipGetLastError();
}

__global__ void k_dense_diag(const double* __restrict__ A, int64_t lda, int64_t n,
                             double* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) d[i] = A[i * lda + i];
}
hipError_t dense_diag(const double* A, int64_t lda, int64_t n, double* diag, hipStream_t s) {
  hipLaunchKernelGGL(k_dense_diag, dim3(cdiv(n, 256)), dim3(256), 0, s, A, lda, n, diag);
  return hipGetLastError();
}

__global__ void k_kron_diag(const double* __restrict__ A, const double* __restrict__ Vp,
                            int64_t na, double* __restrict__ d) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= na * na) return;
  const int64_t i = idx / na, j = idx - i * na;
  d[idx] = A[i * na + i] + A[j * na + j] + Vp[idx];
}
hipError_t kronsum_diag(const double* A, const double* Vp, int64_t na, double* diag,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_kron_diag, dim3(cdiv(na * na, 256)), dim3(256), 0, s, A, Vp, na, diag);
  return hipGetLastError();
}

}  // namespace lobpcg
