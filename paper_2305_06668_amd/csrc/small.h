// Device helpers that the small dense kernels share: lane moves, wave and
// workgroup reductions, the parallel cyclic Jacobi eigensolver.
#pragma once
#include <type_traits>

#include "internal.h"

namespace lobpcg {

constexpr double kEps = 0x1.0p-52;  // double precision machine epsilon
constexpr int kJacobiMaxSweeps = 40;
constexpr int kEigLdsBytes = 152 * 1024;  // dynamic LDS of the eigensolver kernels

__device__ __forceinline__ uint64_t sm64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// index of the wave in its workgroup, in a scalar register
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// LDS writes of one wave visible to the same wave's later reads
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true));
}
// lane L of each row of 16 to the whole row (row_newbcast, the one control that
// the 64-bit DPP move takes)
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x150 + L, 0xF, 0xF, true);
}
// f(integral constant I) for I = B .. E-1
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}
// Sum over the 16 lanes of a row, the same bits in every lane (swap
// neighbours, swap pairs, mirror 8, mirror 16; each step adds the same two
// operands on both partners).
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return v;
}
__device__ __forceinline__ double row_max(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  v = fmax(v, dpp_f64<0x141>(v));
  return fmax(v, dpp_f64<0x140>(v));
}
// (v of this lane's row or of the row beside it in the pair) for N = 16, of
// the wave's lower and upper half for N = 32; the same in all lanes concerned
template <int N>
__device__ __forceinline__ void lane_pair(double v, double& a, double& b) {
  if constexpr (N == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    a = __hiloint2double(h[0], l[0]);
    b = __hiloint2double(h[1], l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    a = __hiloint2double(h[0], l[0]);
    b = __hiloint2double(h[1], l[1]);
  }
}
// Sum (maximum) over the 64 lanes (all active), the same bits in every lane
__device__ __forceinline__ double wave_sum(double v) {
  double a, b;
  lane_pair<16>(row_sum(v), a, b);
  lane_pair<32>(a + b, a, b);
  return a + b;
}
__device__ __forceinline__ double wave_max(double v) {
  double a, b;
  lane_pair<16>(row_max(v), a, b);
  lane_pair<32>(fmax(a, b), a, b);
  return fmax(a, b);
}

// ---------------------------------------------------------------------------
// block-wide helpers (every thread of the block calls them)

__device__ __forceinline__ double blk_reduce_sum_ordered(double v, double* scratch) {
  // scratch: blockDim.x / 64 doubles
  // deterministic: each wave reduces by a fixed xor tree, waves in order
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[w] = v;
  __syncthreads();
  double r = scratch[0];
  for (int i = 1; i < nw; ++i) r += scratch[i];
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------------------
// Parallel cyclic Jacobi on the symmetric n x n matrix A (LDS, stride lda),
// accumulating V (stride ldv, initialised here to I).  Round-robin pairing:
// in round r the pairs are {pp-1, r} and {(r+k) mod (pp-1), (r-k) mod (pp-1)}
// for k = 1 .. pp/2-1, with pp = n rounded up to even (index n is a dummy).
// Two phases per round: (1) one thread per pair computes its rotation from
// the current 2x2 block; (2) every 2x2 block {i0,i1} x {j0,j1} of two pairs
// is rotated in place from both sides by one thread (it is closed under
// J^T A J, so no double buffer is needed), and V's column pairs likewise.
// A rotation is skipped when |a_pq| <= 2^-53 sqrt(|a_pp a_qq|) or
// |a_pq| <= 2^-60 ||A||_F; the sweep loop stops after a sweep without any
// rotation.  Returns the number of sweeps.

// NT: threads of the workgroup.
template <int NT>
__device__ __forceinline__ int blk_jacobi(double* A, int lda, double* V, int ldv, int n, double* cs, int* pr,
                          int* rot_flag, double* scratch) {
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
    const int i = idx / n, j = idx - i * n;
    V[i * ldv + j] = (i == j) ? 1.0 : 0.0;
  }
  double fro = 0.0;
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
    const double v = A[(idx / n) * lda + idx % n];
    fro += v * v;
  }
  fro = sqrt(blk_reduce_sum_ordered(fro, scratch));
  const double abs_tol = 0x1.0p-60 * fro;
  if (n < 2) return 0;
  const int pp = n + (n & 1);
  const int npairs = pp / 2;
  double* cc = cs;            // cos per pair
  double* ss = cs + 64;       // sin per pair
  double* tt = cs + 128;      // tan per pair
  int sweep = 0;
  for (; sweep < kJacobiMaxSweeps; ++sweep) {
    if (threadIdx.x == 0) *rot_flag = 0;
    __syncthreads();
    for (int r = 0; r < pp - 1; ++r) {
      for (int k = threadIdx.x; k < npairs; k += blockDim.x) {
        int i, j;
        if (k == 0) {
          i = pp - 1;
          j = r;
        } else {
          i = r + k;
          if (i >= pp - 1) i -= pp - 1;
          j = r - k;
          if (j < 0) j += pp - 1;
        }
        if (i > j) {
          const int t = i;
          i = j;
          j = t;
        }
        double c = 1.0, sn = 0.0, tn = 0.0;
        if (j < n) {
          const double apq = A[i * lda + j];
          const double app = A[i * lda + i], aqq = A[j * lda + j];
          if (fabs(apq) > 0x1.0p-53 * sqrt(fabs(app * aqq)) && fabs(apq) > abs_tol) {
            const double tau = (aqq - app) / (2.0 * apq);
            tn = (tau >= 0.0) ? 1.0 / (tau + sqrt(1.0 + tau * tau))
                              : -1.0 / (-tau + sqrt(1.0 + tau * tau));
            c = 1.0 / sqrt(1.0 + tn * tn);
            sn = tn * c;
            *rot_flag = 1;
          }
        }
        pr[2 * k] = i;
        pr[2 * k + 1] = j;
        cc[k] = c;
        ss[k] = sn;
        tt[k] = tn;
      }
      __syncthreads();
      // Phase 2: item (ty, tx) of a 32 x 32 grid owns the 2x2 blocks (P, Q)
      // for P in {ty, ty+32}, Q in {tx, tx+32} with P <= Q, and V's column
      // pair Q on the rows ty, ty+32, ty+64; every load of an item is issued
      // before its arithmetic.  The items of a round are independent.
#pragma unroll 1
      for (int it = 0; it < 1024 / NT; ++it) {
      const int tx = threadIdx.x & 31, ty = (threadIdx.x >> 5) + it * (NT / 32);
#pragma unroll
      for (int hq = 0; hq < 2; ++hq) {
        const int Q = tx + 32 * hq;
        if (Q >= npairs) continue;
        const double cQ = cc[Q], sQ = ss[Q], tQ = tt[Q];
        const int j0 = pr[2 * Q], j1 = pr[2 * Q + 1];
        const bool vj1 = j1 < n;
#pragma unroll
        for (int hp = 0; hp < 2; ++hp) {
          const int P = ty + 32 * hp;
          if (P >= npairs || P > Q) continue;
          if (P == Q) {
            if (sQ == 0.0) continue;  // skipped or dummy pair
            const double a01 = A[j0 * lda + j1];
            const double a00 = A[j0 * lda + j0], a11 = A[j1 * lda + j1];
            A[j0 * lda + j0] = a00 - tQ * a01;
            A[j1 * lda + j1] = a11 + tQ * a01;
            A[j0 * lda + j1] = 0.0;
            A[j1 * lda + j0] = 0.0;
            continue;
          }
          const double cP = cc[P], sP = ss[P];
          if (sP == 0.0 && sQ == 0.0) continue;
          const int i0 = pr[2 * P], i1 = pr[2 * P + 1];
          const bool vi1 = i1 < n;
          const double b00 = A[i0 * lda + j0];
          const double b01 = vj1 ? A[i0 * lda + j1] : 0.0;
          const double b10 = vi1 ? A[i1 * lda + j0] : 0.0;
          const double b11 = (vi1 && vj1) ? A[i1 * lda + j1] : 0.0;
          // rows (J^T A): i0' = c i0 - s i1, i1' = s i0 + c i1
          const double t00 = cP * b00 - sP * b10, t01 = cP * b01 - sP * b11;
          const double t10 = sP * b00 + cP * b10, t11 = sP * b01 + cP * b11;
          // columns (A J): j0' = c j0 - s j1, j1' = s j0 + c j1
          const double n00 = cQ * t00 - sQ * t01, n01 = sQ * t00 + cQ * t01;
          const double n10 = cQ * t10 - sQ * t11, n11 = sQ * t10 + cQ * t11;
          A[i0 * lda + j0] = n00;
          A[j0 * lda + i0] = n00;
          if (vj1) {
            A[i0 * lda + j1] = n01;
            A[j1 * lda + i0] = n01;
          }
          if (vi1) {
            A[i1 * lda + j0] = n10;
            A[j0 * lda + i1] = n10;
          }
          if (vi1 && vj1) {
            A[i1 * lda + j1] = n11;
            A[j1 * lda + i1] = n11;
          }
        }
        if (sQ != 0.0) {
          // rows ty, ty + 32, ty + 64 (clamped reads, guarded writes)
          const int r0 = ty, r1 = ty + 32, r2 = ty + 64;
          const int q1 = (r1 < n) ? r1 : r0, q2 = (r2 < n) ? r2 : r0;
          const double a0 = V[r0 * ldv + j0], b0 = V[r0 * ldv + j1];
          const double a1 = V[q1 * ldv + j0], b1 = V[q1 * ldv + j1];
          const double a2 = V[q2 * ldv + j0], b2 = V[q2 * ldv + j1];
          if (r0 < n) {
            V[r0 * ldv + j0] = cQ * a0 - sQ * b0;
            V[r0 * ldv + j1] = sQ * a0 + cQ * b0;
          }
          if (r1 < n) {
            V[r1 * ldv + j0] = cQ * a1 - sQ * b1;
            V[r1 * ldv + j1] = sQ * a1 + cQ * b1;
          }
          if (r2 < n) {
            V[r2 * ldv + j0] = cQ * a2 - sQ * b2;
            V[r2 * ldv + j1] = sQ * a2 + cQ * b2;
          }
        }
      }
      }
      __syncthreads();
    }
    const int any = *rot_flag;
    __syncthreads();
    if (!any) break;
    // stop without a confirming sweep when no pair would rotate any more
    if (threadIdx.x == 0) *rot_flag = 0;
    __syncthreads();
    for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
      const int i = idx / n, j = idx - i * n;
      if (j <= i) continue;
      const double apq = A[i * lda + j];
      if (fabs(apq) > 0x1.0p-53 * sqrt(fabs(A[i * lda + i] * A[j * lda + j])) && fabs(apq) > abs_tol)
        *rot_flag = 1;
    }
    __syncthreads();
    const int more = *rot_flag;
    __syncthreads();
    if (!more) break;
  }
  return sweep + 1;
}

// evals ascending (ties by index) -> perm[rank] = index
__device__ __forceinline__ void blk_sort_evals(const double* A, int lda, int n, int* perm) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double li = A[i * lda + i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double lj = A[j * lda + j];
      if (lj < li || (lj == li && j < i)) ++rank;
    }
    perm[rank] = i;
  }
  __syncthreads();
}

}  // namespace lobpcg
