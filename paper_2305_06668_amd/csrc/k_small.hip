// Small dense fp64 linear algebra of the LOBPCG step, one workgroup each,
// everything resident in LDS (gfx950: 160 KB per workgroup):
//   * cyclic Jacobi eigensolver in parallel (round-robin) order for the
//     p x p Rayleigh-Ritz matrix, p <= 96 (Alg. 1, "solve a u = lambda u";
//     the paper calls LAPACK dsyev, Sec. 3.1);
//   * shifted Cholesky of an overlap matrix (Sec. 3.2: retry with
//     alpha * eps * ||X|| added to the diagonal, alpha = 100, 1000, ...);
//   * the implicit P coefficients u_p = ortho(u_x[:, act] - E[:, act]; u_x)
//     in R^p (Alg. 1 and the "Basis selection" paragraph of Sec. 3.1);
//   * the controller of ortho(W; Y) on n-vectors (Alg. 2 inside Alg. 3): it
//     reads the overlap G = [Y W]^T W of the current W and emits the small
//     coefficient matrix that the streaming kernel applies next.
#include <type_traits>

#include "internal.h"

namespace lobpcg {

constexpr double kEps = 0x1.0p-52;  // double precision machine epsilon
constexpr double kShiftAlpha0 = 100.0;
constexpr double kShiftGrowth = 10.0;
constexpr int kShiftRetries = 20;
constexpr int kJacobiMaxSweeps = 40;

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
// the 64-bit DPP move (row_newbcast is the one control it takes)
extern "C" __device__ long lobpcg_update_dpp_i64(long old, long src, int ctrl, int row_mask, int bank_mask,
                                                 bool bound_ctrl) __asm("llvm.amdgcn.update.dpp.i64");
// lane L of each row of 16 to the whole row
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
  const long x = __double_as_longlong(v);
  return __longlong_as_double(lobpcg_update_dpp_i64(x, x, 0x150 + L, 0xF, 0xF, true));
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

// 1 / q and 1 / sqrt(x) to 1 ulp: the hardware estimate (2^-23 or better)
// and two Newton steps.  q, x finite and not 0, x > 0.
__device__ __forceinline__ double rcp2(double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(r, fma(-q, r, 1.0), r);
  return fma(r, fma(-q, r, 1.0), r);
}
__device__ __forceinline__ double rsq2(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// Cholesky of a 16 x 16 matrix by one wave, each row of 16 lanes with a copy
// of its own: lane l holds matrix row l % 16 in g (g[c] read for c <= row).
// An n x n matrix (n < 16) comes padded with the identity.  The next pivot
// is a lane broadcast, a reciprocal square root and one update away from the
// last, which is the chain that bounds it: 1.5 us with the broadcasts as DPP
// moves, 8.6 us with a rounded root and division per column and lane shuffles
// through LDS.  On return g holds L and inv the reciprocals of its diagonal.
// False (uniform) when a pivot was not > 0 or not finite.
__device__ __forceinline__ bool chol16_rows(double (&g)[16], int n, double (&inv)[16]) {
  const int row = threadIdx.x & 15;
  bool ok = true;
  auto column = [&](auto K) {
    constexpr int k = K;
    const double piv = row_bcast<k>(g[k]);
    ok = ok && piv > 0.0 && piv < INFINITY;
    const double y = rsq2(piv);
    inv[k] = y;
    const double lk = ((row == k) ? piv : g[k]) * y;
    g[k] = lk;
    const double nlk = -lk;
    static_for<k + 1, 16>([&](auto C) { g[C] = fma(row_bcast<C>(lk), nlk, g[C]); });
  };
  static_for<0, 16>([&](auto K) { inv[K] = 1.0; });
  static_for<0, 4>(column);
  if (n > 4) static_for<4, 8>(column);
  if (n > 8) static_for<8, 16>(column);
  return __builtin_amdgcn_readfirstlane(ok) != 0;
}

// Rows of X (p x n, n <= 16) times L^-T, thread i taking row i, with L and
// inv as chol16_rows left them in this thread's row of 16 lanes
__device__ __forceinline__ void trsm16_rows(double* X, int ldx, int p, int n, const double (&g)[16],
                                            const double (&inv)[16]) {
  const int i = threadIdx.x;
  double z[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) z[c] = (c < n && i < p) ? X[i * ldx + c] : 0.0;
  auto column = [&](auto C) {
    constexpr int c = C;
    z[c] *= inv[c];
    const double nz = -z[c];
    static_for<c + 1, 16>([&](auto K) { z[K] = fma(row_bcast<K>(g[c]), nz, z[K]); });
  };
  static_for<0, 4>(column);
  if (n > 4) static_for<4, 8>(column);
  if (n > 8) static_for<8, 16>(column);
  if (i < p) {
#pragma unroll
    for (int c = 0; c < 16; ++c)
      if (c < n) X[i * ldx + c] = z[c];
  }
}

// ---------------------------------------------------------------------------
// block-wide helpers (every thread of the block calls them)

__device__ __forceinline__ double blk_reduce_max(double v, double* scratch) {
  // scratch: blockDim.x / 64 doubles
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[w] = v;
  __syncthreads();
  double r = scratch[0];
  for (int i = 1; i < nw; ++i) r = fmax(r, scratch[i]);
  __syncthreads();
  return r;
}

__device__ __forceinline__ double blk_reduce_sum_ordered(double v, double* scratch) {
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

// scale columns of X (n x q) to unit norm, 16 lanes per column; exact-zero
// columns are replaced by SplitMix64 columns (entry i of column j:
// splitmix64(seed + j n + i)).
__device__ __forceinline__ void blk_normalize(double* X, int ldx, int n, int q, int* zeros) {
  const int l = threadIdx.x & 15;
  for (int j = threadIdx.x >> 4; j < q; j += blockDim.x >> 4) {
    double s = 0.0;
    for (int r = l; r < n; r += 16) s = fma(X[r * ldx + j], X[r * ldx + j], s);
    s = row_sum(s);
    if (s == 0.0) {  // uniform over the 16 lanes
      for (int r = l; r < n; r += 16) {
        const uint64_t z = sm64(kZeroColumnSeed + (uint64_t)j * (uint64_t)n + (uint64_t)r);
        const double x = (double)(z >> 11) * 0x1.0p-53 - 0.5;
        X[r * ldx + j] = x;
        s = fma(x, x, s);
      }
      s = row_sum(s);
      if (l == 0) atomicAdd(zeros, 1);
    }
    const double inv = rsq2(s);
    for (int r = l; r < n; r += 16) X[r * ldx + j] *= inv;
  }
  __syncthreads();
}

// Cholesky L L^T = M + shift I (lower, n x n; the strict upper part of L is
// zeroed); returns true on success.  Breaks down when a pivot is not > 0 (NaN
// included), like LAPACK potrf.  Every thread calls it and M must be complete
// on entry.  Wave 0 alone factors (REG and n <= 16: in registers, else column
// by column in LDS with wave-level syncs) while the other waves wait at the
// closing barriers: two workgroup barriers per factorization.
template <bool REG = true>
__device__ __forceinline__ bool blk_chol(const double* M, int ldm, int n, double shift, double* L, int ldl,
                         int* flag) {
  if (REG && threadIdx.x < 64 && n <= 16) {
    const int r = threadIdx.x & 15;
    double g[16], inv[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
      g[c] = (r < n && c <= r) ? M[r * ldm + c] + (r == c ? shift : 0.0) : (r == c ? 1.0 : 0.0);
    const bool ok = chol16_rows(g, n, inv);
    if ((int)threadIdx.x < n) {
#pragma unroll
      for (int c = 0; c < 16; ++c)
        if (c < n) L[r * ldl + c] = (c <= r) ? g[c] : 0.0;
    }
    if (threadIdx.x == 0) *flag = ok ? 0 : 1;
  } else if (threadIdx.x < 64) {
    const int l = threadIdx.x;
    for (int idx = l; idx < n * n; idx += 64) {
      const int i = idx / n, j = idx - i * n;
      L[i * ldl + j] = (j <= i) ? (M[i * ldm + j] + (i == j ? shift : 0.0)) : 0.0;
    }
    int bad = 0;
    wave_sync();
    for (int j = 0; j < n; ++j) {
      const double d = L[j * ldl + j];
      if (!(d > 0.0)) {  // uniform across the wave
        bad = 1;
        break;
      }
      const double ljj = sqrt(d);
      if (l == 0) L[j * ldl + j] = ljj;
      for (int i = j + 1 + l; i < n; i += 64) L[i * ldl + j] /= ljj;
      wave_sync();
      const int rem = n - j - 1;
      for (int idx = l; idx < rem * rem; idx += 64) {
        const int i = j + 1 + idx / rem, k = j + 1 + idx % rem;
        if (k <= i) L[i * ldl + k] -= L[i * ldl + j] * L[k * ldl + j];
      }
      wave_sync();
    }
    if (l == 0) *flag = bad;
  }
  __syncthreads();
  const bool ok = (*flag == 0);
  __syncthreads();  // the flag is rewritten by the next call
  return ok;
}

struct ShiftCount {
  int factorizations, failed, shifted, svqb;
};

// Sec. 3.2 / Alg. 2: plain Cholesky, then shifts alpha*eps*||X||_F with
// ||X||_F = sqrt(trace M), alpha = 100, x10 per retry.
template <bool REG = true>
__device__ __forceinline__ bool blk_shifted_chol(const double* M, int ldm, int n, double* L, int ldl, int* flag,
                                 ShiftCount* c, int retries = kShiftRetries) {
  if (threadIdx.x == 0) c->factorizations++;
  if (blk_chol<REG>(M, ldm, n, 0.0, L, ldl, flag)) return true;
  if (threadIdx.x == 0) c->failed++;
  double tr = 0.0;
  for (int i = 0; i < n; ++i) tr += M[i * ldm + i];
  const double normx = sqrt(fmax(tr, 0.0));
  double alpha = kShiftAlpha0;
  for (int t = 0; t < retries; ++t) {
    if (threadIdx.x == 0) c->factorizations++;
    if (blk_chol<REG>(M, ldm, n, alpha * kEps * normx, L, ldl, flag)) {
      if (threadIdx.x == 0) c->shifted++;
      return true;
    }
    if (threadIdx.x == 0) c->failed++;
    alpha *= kShiftGrowth;
  }
  return false;
}

// Linv = L^-1 (lower), one column per thread by forward substitution.
__device__ __forceinline__ void blk_tri_inv(const double* L, int ldl, int n, double* Li, int ldi) {
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    for (int i = 0; i < n; ++i) {
      if (i < j) {
        Li[i * ldi + j] = 0.0;
        continue;
      }
      double s = (i == j) ? 1.0 : 0.0;
      for (int k = j; k < i; ++k) s -= L[i * ldl + k] * Li[k * ldi + j];
      Li[i * ldi + j] = s / L[i * ldl + i];
    }
  }
  __syncthreads();
}

// X (n x q) <- X L^-T, one row per thread: z_j = (x_j - sum_{k<j} z_k L_jk) / L_jj
__device__ __forceinline__ void blk_trsm_rt(double* X, int ldx, int n, int q, const double* L, int ldl) {
  for (int r = threadIdx.x; r < n; r += blockDim.x) {
    for (int j = 0; j < q; ++j) {
      double s = X[r * ldx + j];
      for (int k = 0; k < j; ++k) s -= X[r * ldx + k] * L[j * ldl + k];
      X[r * ldx + j] = s / L[j * ldl + j];
    }
  }
  __syncthreads();
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

// Workspace of the Jacobi sweeps besides A and V
struct JacobiLds {
  double cs[3 * 64];
  double scratch[16];
  int pr[2 * 64];
  int perm[128];
  int flags[8];
};

// sym(a) into A (stride lda), scaled by ds[i] ds[j] from both sides
__device__ __forceinline__ void load_sym(const double* a, int p, const double* ds, double* A, int lda) {
  for (int idx = threadIdx.x; idx < p * p; idx += blockDim.x) {
    const int i = idx / p, j = idx - i * p;
    A[i * lda + j] = 0.5 * (a[i * p + j] + a[j * p + i]) * (ds[i] * ds[j]);
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Lowest nev eigenpairs of a symmetric p x p matrix by the tridiagonal
// route (the Rayleigh-Ritz solve of Alg. 1; the paper calls LAPACK for it,
// Sec. 3.1), by one workgroup of four waves:
//   1. Householder reduction A = Q T Q^T: reflector k,
//      H_k = I - beta_k v_k v_k^T, maps column k below the diagonal to
//      alpha_k e_{k+1} (Q = H_0 H_1 ... H_{p-2}, the last one I);
//   2. the nev lowest eigenvalues of T by multisection on Sturm counts,
//      G points per eigenvalue and round;
//   3. their vectors by block inverse iteration: a solve with the
//      partial-pivoting LU of T - lambda_j I from a SplitMix64 start
//      (pivots below eps ||T|| raised to eps ||T||, one thread per vector),
//      Cholesky-QR of the nev vectors, a second solve;
//   4. back-transformation u = Q z, 16 lanes per vector;
//   5. Cholesky-QR, twice, of the nev vectors.
// Inverse iteration returns the vectors of a cluster of close or repeated
// eigenvalues as independent mixtures of the cluster's eigenvectors, which
// drift towards each other with further solves; orthonormalising them in
// ascending order between and after the solves keeps them an orthonormal
// eigenbasis of the cluster.  Cholesky-QR goes by panels of 16 columns, each
// made orthogonal to the ones before it first.
// What bounds it is the latency of dependent fp64 steps, not their number,
// so every phase is laid out for a short chain: the matrix of phase 1 and
// the factors of phase 5 stay in registers, four waves make a barrier cheap
// (16 waves bring it no more arithmetic worth having, and leave each 128
// registers), every function is inlined (a call would turn its LDS accesses
// into flat ones and its uniform arguments into vector registers), reciprocals and square roots are the hardware's estimate with
// two Newton steps (1 ulp; a correctly rounded division is about twice as
// many dependent operations), small products run on the fp64 MFMA.
// Returns false when a Cholesky-QR breaks down; the callers then reload A
// and run Jacobi.

constexpr int kEigLdsBytes = 152 * 1024;  // dynamic LDS of the eigensolver kernels
constexpr int kEigThreads = 256;

typedef double dd2 __attribute__((ext_vector_type(2)));

// LDS layout of the tridiagonal path, in doubles.  `work` is where a caller
// may lay its own data over everything but Z and ev once the vectors are
// done.  The reduction's vectors and the LU of the inverse iteration share
// `lu`.  Z and the LU have rows for p rounded up to 8.
struct TriLayout {
  int ldz, nb;
  int Z, ev, d, e, beta, work, de, vref, orth, lu, total;
};
constexpr int kTrans = 16 * 17;  // one wave's 16 x 16 transpose
constexpr int kRedScratch = 128 + 4 * 128;
// reflectors: rows of 64 up to p = 64 (zeros in front and behind), packed above
__host__ __device__ inline int ref_doubles(int p) { return p <= 64 ? 64 * p : p * (p - 1) / 2; }
__host__ __device__ inline TriLayout tri_layout(int p, int nev) {
  TriLayout t;
  const int p8 = (p + 7) & ~7;
  t.ldz = nev | 1;
  int o = 0;
  t.Z = o; o += p8 * t.ldz;
  t.ev = o; o += nev;
  t.d = o; o += p8 + 1;
  t.e = o; o += p8 + 1;
  t.beta = o; o += p;
  o += o & 1;
  t.work = o;
  t.de = o; o += 2 * (p + 16);
  t.vref = o; o += ref_doubles(p);
  t.orth = o; o += 4 * kTrans + (nev > 16 ? (nev - 1) / 16 * 16 * 17 : 0);
  t.lu = o;
  const int avail = kEigLdsBytes / 8 - o;
  int nb = avail / (3 * p8);  // U0^-1, U1, multipliers
  if (nb > nev) nb = nev;
  t.nb = nb;
  const int lu = 3 * p8 * nb;
  t.total = o + (lu > kRedScratch ? lu : kRedScratch);
  return t;
}
// the path runs for every p the kernels take, also with all vectors wanted
static_assert(kEigLdsBytes / 8 > 96 * 97 + 4 * 98 + 2 * 112 + 96 * 95 / 2 + 4 * kTrans + 80 * 17 + kRedScratch &&
                  kEigLdsBytes / 8 > 64 * 65 + 4 * 66 + 2 * 80 + 64 * 64 + 4 * kTrans + 48 * 17 + kRedScratch,
              "LDS of the largest eigensolves");

// offset of reflector k (its entries k+1 .. p-1) in the packed store
__device__ __forceinline__ int ref_off(int p, int k) { return k * (p - 1) - k * (k - 1) / 2; }

// Householder reduction of sym(a) scaled by ds from both sides.  Lane l of
// wave w keeps, in registers, rows l (and l + 64: H = 2) of the columns
// c = w (mod 4), slot by slot; every four steps each wave takes its next slot
// out as `cur`, the pivot of one of those steps, and moves the rest down.
// Per step the pivot's wave forms the reflector (one wave sum, a reciprocal
// square root, a reciprocal) and hands it out through LDS (barrier); every
// wave takes its columns' part of A v and exchanges the parts (barrier); each
// then has p = beta A v, K = beta / 2 p^T v and w = p - K v in all its lanes
// and updates A -= v w^T + w v^T.  The v and w of its own columns a wave reads
// from its lanes (a broadcast from LDS costs a whole wave's worth of its
// return path, four waves' worth per step).  Rows above the pivot only see
// reflections and are not read any more; a zero reflector (beta = 0) changes
// nothing.  One wave per SIMD, so the instruction count of a step is its time:
// two barriers and about 2100 cycles, where the trailing matrix in LDS under 16 waves took
// three barriers and 3500 (p = 48: 67 us, now 42).
template <int H, int NJ>
__device__ __forceinline__ void reg_tridiag(const double* __restrict__ a, int p, const double* ds, double* d,
                                            double* e, double* beta, double* vref, double* scr) {
  double* vlin = scr;         // 64 H (H = 2; else the reflector's row of vref)
  double* part = vlin + 128;  // [wave][128]
  const int lane = threadIdx.x & 63, wave = wave_id();
  if (H == 2 && threadIdx.x < 128) vlin[threadIdx.x] = 0.0;
  double A[H][NJ], cur[H];
#pragma unroll
  for (int h = 0; h < H; ++h)
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const int i = lane + 64 * h, c = 4 * jj + wave;
      A[h][jj] = (i < p && c < p) ? 0.5 * (a[i * p + c] + a[c * p + i]) * (ds[i] * ds[c]) : 0.0;
    }
  __syncthreads();
  const int nslot = (p + 3) >> 2;
  // lane c of x[] (c uniform); 0 past the lanes, where a chunk's last slots
  // may lie with one row per lane and more than 52 of them (their columns are
  // empty and stay so)
  auto at = [](const double (&x)[H], int c) {
    if (H == 1 && 4 * NJ > 52 && c > 63) return 0.0;
    return (H == 1 || c < 64) ? readlane_f64(x[0], c & 63) : readlane_f64(x[H - 1], c & 63);
  };
  for (int o = 0; o < nslot; ++o) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      cur[h] = A[h][0];
#pragma unroll
      for (int jj = 0; jj + 1 < NJ; ++jj) A[h][jj] = A[h][jj + 1];
      A[h][NJ - 1] = 0.0;
    }
    const int nrem = nslot - 1 - o;  // slots behind cur
    for (int w4 = 0; w4 < 4; ++w4) {
      const int k = 4 * o + w4, k1 = k + 1;
      if (k1 >= p) {
        if (k < p && wave == w4) {
          // the last column: its diagonal entry
#pragma unroll
          for (int h = 0; h < H; ++h)
            if (lane + 64 * h == k) d[k] = cur[h];
        }
        break;
      }
      if (wave == w4) {
        double tail = 0.0;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const double t = (lane + 64 * h > k1) ? cur[h] : 0.0;
          tail = fma(t, t, tail);
        }
        const double x0 = at(cur, k), x1 = at(cur, k1);
        tail = wave_sum(tail);
        double alpha = x1, b = 0.0;
        if (tail > 0.0) {
          const double s2 = fma(x1, x1, tail);
          const double y = rsq2(s2);
          double nrm = s2 * y;
          nrm = fma(0.5 * y, fma(-nrm, nrm, s2), nrm);
          alpha = (x1 >= 0.0) ? -nrm : nrm;
          b = rcp2(nrm * (nrm + fabs(x1)));  // 2 / v^T v for v = x - alpha e_1
        }
        const double v1 = x1 - alpha;
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int i = lane + 64 * h;
          const double v = (i > k1) ? cur[h] : ((i == k1) ? v1 : 0.0);
          if (H == 1) {
            vref[64 * k + i] = v;
          } else if (i < p) {
            vlin[i] = v;
            if (i > k) vref[ref_off(p, k) + i - k1] = v;
          }
        }
        if (lane == 0) {
          d[k] = x0;
          e[k] = alpha;
          beta[k] = b;
        }
      }
      __syncthreads();
      // the part of A v that this wave's columns give
      const double b = beta[k];
      const double* vrow = (H == 1) ? vref + 64 * k : vlin;
      double vi[H], vj[NJ], acc[H][2];
#pragma unroll
      for (int h = 0; h < H; ++h) vi[h] = vrow[lane + 64 * h];
      const int c0 = 4 * o + wave;  // cur's column; slot jj holds c0 + 4 (jj + 1)
      const double vc = at(vi, c0);
#pragma unroll
      for (int h = 0; h < H; ++h) {
        acc[h][0] = cur[h] * vc;
        acc[h][1] = 0.0;
      }
#pragma unroll
      for (int c4 = 0; c4 < NJ; c4 += 4)
        if (c4 < nrem) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            vj[c4 + u] = at(vi, c0 + 4 * (c4 + u + 1));
#pragma unroll
            for (int h = 0; h < H; ++h) acc[h][u & 1] = fma(A[h][c4 + u], vj[c4 + u], acc[h][u & 1]);
          }
        }
#pragma unroll
      for (int h = 0; h < H; ++h) part[wave * 128 + lane + 64 * h] = acc[h][0] + acc[h][1];
      __syncthreads();
      double wi[H], kp = 0.0;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const double* q = part + lane + 64 * h;
        wi[h] = b * ((q[0] + q[128]) + (q[256] + q[384]));
        kp = fma(wi[h], vi[h], kp);
      }
      const double nK = -0.5 * b * wave_sum(kp);
#pragma unroll
      for (int h = 0; h < H; ++h) wi[h] = fma(nK, vi[h], wi[h]);
      const double wc = at(wi, c0);
#pragma unroll
      for (int h = 0; h < H; ++h) cur[h] = fma(-wi[h], vc, fma(-vi[h], wc, cur[h]));
#pragma unroll
      for (int c4 = 0; c4 < NJ; c4 += 4)
        if (c4 < nrem) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double wj = at(wi, c0 + 4 * (c4 + u + 1));
#pragma unroll
            for (int h = 0; h < H; ++h)
              A[h][c4 + u] = fma(-wi[h], vj[c4 + u], fma(-vi[h], wj, A[h][c4 + u]));
          }
        }
    }
  }
  __syncthreads();
}

// Sturm count of T - x I: the number of sign changes in p_0 = 1,
// p_1 = d_0 - x, p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1} (the leading
// minors), one fused multiply-add per dependent step where the pivots'
// quotient form has a reciprocal and two.  de[i] = (d_i, e_{i-1}^2) for ||T||
// in [1, 2), with e^2 raised to 2^-120 (a change of T below its rounding): a
// zero minor is then followed by a nonzero one of the other sign, one sign
// change whichever sign the zero carries.  A step multiplies the pair by at
// most 2^4 and at least about 2^-60; a power of two brings it back to 1 every
// 8 steps.  de is padded with steps that change no sign, and the operands of
// the next eight steps are loaded ahead.
__device__ __forceinline__ int sturm_count(const dd2* __restrict__ de, int p, double x) {
  const dd2 t0 = de[0];
  double p0 = 1.0, p1 = t0[0] - x;
  uint32_t c = (uint32_t)__double2hiint(p1) >> 31;
  dd2 t[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    t[u] = de[1 + u];
    asm("" : "+v"(t[u]));  // (else the compiler folds the two loads into one at the loop's top)
  }
  for (int i = 1; i < p; i += 8) {
    dd2 tn[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) tn[u] = de[i + 8 + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double pn = fma(t[u][0] - x, p1, -(t[u][1] * p0));
      c += (uint32_t)(__double2hiint(pn) ^ __double2hiint(p1)) >> 31;
      p0 = p1;
      p1 = pn;
    }
    const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
    p0 = __builtin_amdgcn_ldexp(p0, -ex);
    p1 = __builtin_amdgcn_ldexp(p1, -ex);
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = tn[u];
  }
  return (int)c;
}

// Eigenvalues 0 .. nev-1 (ascending) of T into ev, G lanes to each: the
// largest power of two (64 at most) with one point per thread.  More points
// per thread shorten the search by less than they add to the count loop,
// which one wave per SIMD runs at its instruction rate.  Every thread calls
// it.
__device__ __forceinline__ void blk_multisection(const dd2* de, int p, int nev, double gl, double gu, double tnorm,
                                                 double* ev) {
  int G = 64;
  while (G > 1 && G * nev > kEigThreads) G >>= 1;
  const int lane = threadIdx.x & 63;
  const int t = lane & (G - 1), gi = (int)threadIdx.x / G;
  const uint64_t gmask = (G == 64) ? ~0ull : (((1ull << G) - 1ull) << (lane & ~(G - 1)));
  const double inv = 1.0 / (double)(G + 1), tp = (double)(t + 1);
  for (int j0 = 0; j0 < nev; j0 += kEigThreads / G) {
    const int j = j0 + gi;
    bool act = j < nev;
    double lo = gl, hi = gu;
    for (int round = 0; round < 256; ++round) {
      const double w = hi - lo;
      act = act && !(w <= 2.0 * kEps * fmax(fabs(lo), fabs(hi)) || w <= kEps * tnorm);
      if (__ballot(act) == 0) break;
      const double h = w * inv;
      const int c = sturm_count(de, p, fma(tp, h, lo));
      const int k = __popcll(__ballot(c <= j) & gmask);
      const double nlo = (k > 0) ? fma((double)k, h, lo) : lo;
      const double nhi = (k < G) ? fma((double)(k + 1), h, lo) : hi;
      act = act && !(nlo == lo && nhi == hi);
      if (act) {
        lo = nlo;
        hi = nhi;
      }
    }
    if (t == 0 && j < nev) ev[j] = lo + 0.5 * (hi - lo);
  }
}

// One inverse-iteration solve of (T - lam I) z = Z[:, j], thread t of nb.
// FACTOR builds the LU (partial pivoting by selects, so that lanes that swap
// and lanes that do not take the same steps) and keeps U0^-1, U1 and the
// multipliers in LDS, the swaps as bits in sw0, sw1: U2 is e_{i+1} after a
// swap, 0 otherwise.  Rows p .. p8-1 continue T by the identity (d = lam + 1,
// e = 0; zero in Z), so that the rows go by eights without a branch, their
// operands loaded ahead of the dependent chain.
template <bool FACTOR>
__device__ __forceinline__ void tri_invit_solve(const double* __restrict__ d, const double* __restrict__ e, int p,
                                                double lam, double tol, double* __restrict__ Z, int ldz, int j,
                                                double* __restrict__ U0, double* __restrict__ U1,
                                                double* __restrict__ LM, int nb, uint64_t& sw0, uint64_t& sw1) {
  const int p8 = (p + 7) & ~7;
  double y = Z[j];
  double c0 = d[0] - lam, c1 = e[0];
  if (FACTOR) sw0 = sw1 = 0;
  for (int i0 = 0; i0 < p8; i0 += 8) {
    // step i eliminates row i + 1; the last chunk's last step meets row p8,
    // which is again one of the identity
    double bz[8], dn[8], en[9], lm[8];
    const bool lastc = i0 + 8 == p8;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u;
      if (u < 7) bz[u] = Z[(i + 1) * ldz + j];
      else bz[u] = lastc ? 0.0 : Z[(i + 1) * ldz + j];
      if (FACTOR) {
        dn[u] = (i + 1 < p) ? d[i + 1] - lam : 1.0;
        en[u] = e[i];
      } else {
        lm[u] = LM[i * nb];
      }
    }
    if (FACTOR) en[8] = e[i0 + 8];
    uint32_t m = 0;
    if (!FACTOR) m = (uint32_t)(((i0 < 64) ? sw0 : sw1) >> (i0 & 63));
    double zo[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      bool s;
      double li;
      if (FACTOR) {
        const double ei = en[u];
        s = fabs(c0) < fabs(ei);
        double piv = s ? ei : c0;
        piv = (fabs(piv) < tol) ? copysign(tol, piv) : piv;
        const double r = rcp2(piv);
        li = (s ? c0 : ei) * r;
        const double u1 = s ? dn[u] : c1;
        U0[(i0 + u) * nb] = r;
        U1[(i0 + u) * nb] = u1;
        LM[(i0 + u) * nb] = li;
        m |= s ? (1u << u) : 0u;
        c0 = fma(-li, u1, s ? c1 : dn[u]);
        c1 = s ? -li * en[u + 1] : en[u + 1];
      } else {
        s = (m >> u) & 1;
        li = lm[u];
      }
      const double zi = s ? bz[u] : y;
      zo[u] = zi;
      y = fma(-li, zi, s ? y : bz[u]);
    }
    if (FACTOR) {
      if (i0 < 64) sw0 |= (uint64_t)m << i0;
      else sw1 |= (uint64_t)m << (i0 - 64);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) Z[(i0 + u) * ldz + j] = zo[u];
  }
  // (the scale of z is left to the Cholesky-QR)
  double z1 = 0.0, z2 = 0.0;
  for (int i0 = p8 - 8; i0 >= 0; i0 -= 8) {
    double zr[8], u0[8], u1[8], u2[8];
    const uint32_t m = (uint32_t)(((i0 < 64) ? sw0 : sw1) >> (i0 & 63));
#pragma unroll
    for (int u = 7; u >= 0; --u) {
      const int i = i0 + u;
      zr[u] = Z[i * ldz + j];
      u0[u] = U0[i * nb];
      u1[u] = U1[i * nb];
      u2[u] = ((m >> u) & 1) ? e[i + 1] : 0.0;
    }
#pragma unroll
    for (int u = 7; u >= 0; --u) {
      const double zi = fma(-u1[u], z1, fma(-u2[u], z2, zr[u])) * u0[u];
      zr[u] = zi;
      z2 = z1;
      z1 = zi;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) Z[(i0 + u) * ldz + j] = zr[u];
  }
}

// ---- small products on the fp64 MFMA 16x16x4 -------------------------------
// Lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator register
// r is row 4 r + l / 16, column l % 16.
__device__ __forceinline__ d4 mma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// One 16 x 16 tile of A^T B (A: K x m, B: K x n), by one wave
__device__ __forceinline__ d4 tile_tn(const double* A, int lda, int i0, int m, const double* B, int ldb, int j0,
                                      int n, int K) {
  const int g = (threadIdx.x & 63) >> 4, r = threadIdx.x & 15;
  const bool vi = i0 + r < m, vj = j0 + r < n;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < K; k0 += 16) {
    double av[4], bv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + 4 * u + g;
      av[u] = (vi && k < K) ? A[k * lda + i0 + r] : 0.0;
      bv[u] = (vj && k < K) ? B[k * ldb + j0 + r] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = mma64(av[u], bv[u], acc);
  }
  return acc;
}
// C (m x n) = A^T B by the workgroup's waves; ends with a barrier
__device__ __forceinline__ void blk_gemm_tn(const double* A, int lda, const double* B, int ldb, int K, int m,
                                            int n, double* C, int ldc) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int tm = (m + 15) >> 4, tn = (n + 15) >> 4;
  for (int t = wave_id(); t < tm * tn; t += blockDim.x >> 6) {
    const int i0 = 16 * (tn == 1 ? t : t / tn), j0 = tn == 1 ? 0 : 16 * (t % tn);
    const d4 acc = tile_tn(A, lda, i0, m, B, ldb, j0, n, K);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 4 * q + g;
      if (i < m && j0 + r < n) C[i * ldc + j0 + r] = acc[q];
    }
  }
  __syncthreads();
}
// X (n x q) -= Y (n x K) C (K x q) by the workgroup's waves; ends with a barrier
__device__ __forceinline__ void blk_sub_mm(double* X, int ldx, const double* Y, int ldy, const double* C, int ldc,
                                           int n, int K, int q) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int tm = (n + 15) >> 4, tn = (q + 15) >> 4;
  for (int t = wave_id(); t < tm * tn; t += blockDim.x >> 6) {
    const int i0 = 16 * (tn == 1 ? t : t / tn), j0 = tn == 1 ? 0 : 16 * (t % tn);
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < K; k0 += 16) {
      double av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + 4 * u + g;
        av[u] = (i0 + r < n && k < K) ? Y[(i0 + r) * ldy + k] : 0.0;
        bv[u] = (j0 + r < q && k < K) ? C[k * ldc + j0 + r] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = mma64(av[u], bv[u], acc);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = i0 + 4 * c + g;
      if (i < n && j0 + r < q) X[i * ldx + j0 + r] -= acc[c];
    }
  }
  __syncthreads();
}

// Row l % 16 of the Gram P^T P (p x n, n <= 16), padded with the identity, in
// every lane of the wave; tr: the wave's transpose area.
__device__ __forceinline__ void gram16_rows(const double* P, int ldp, int p, int n, double* tr, double (&g)[16]) {
  const int lane = threadIdx.x & 63, gq = lane >> 4, r = lane & 15;
  const d4 acc = tile_tn(P, ldp, 0, n, P, ldp, 0, n, p);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = 4 * q + gq;
    tr[i * 17 + r] = (i == r && i >= n) ? 1.0 : acc[q];
  }
  wave_sync();
#pragma unroll
  for (int c = 0; c < 16; ++c) g[c] = tr[r * 17 + c];
  wave_sync();
}

// Z (p x n, stride ldz) <- orthonormal columns: by panels of 16, each made
// orthogonal to the panels before it, then Cholesky-QR.  Every wave forms the
// panel's Gram and factor itself (the same bits), so that the only barriers
// are around the writes of Z.  scr: tri_layout's `orth`.  False (uniform) on
// breakdown.  Every thread calls it; ends with a barrier.
__device__ __forceinline__ bool blk_cholqr(double* Z, int ldz, int p, int n, double* scr) {
  double* tr = scr + wave_id() * kTrans;
  double* C = scr + 4 * kTrans;
  for (int j0 = 0; j0 < n; j0 += 16) {
    const int nb = min(16, n - j0);
    double* P = Z + j0;
    if (j0 > 0) {
      blk_gemm_tn(Z, ldz, P, ldz, p, j0, nb, C, 17);
      blk_sub_mm(P, ldz, Z, ldz, C, 17, p, j0, nb);
    }
    double g[16], inv[16];
    gram16_rows(P, ldz, p, nb, tr, g);
    const bool ok = chol16_rows(g, nb, inv);
    __syncthreads();  // every wave has read the panel
    if (!ok) return false;
    trsm16_rows(P, ldz, p, nb, g, inv);
    __syncthreads();
  }
  return true;
}

// u = H_0 H_1 ... H_{p-2} z for the columns of Z: 16 lanes per vector, NT
// rows per lane, four vectors per wave; reflector k - 1 is loaded while
// reflector k is applied (PACK: from the packed store)
template <int NT, bool PACK>
__device__ __forceinline__ void blk_backtransform(double* Z, int ldz, int p, int nev, const double* vref,
                                                  const double* beta) {
  const int lane = threadIdx.x & 63, s = lane & 15;
  for (int jb = 0; jb < nev; jb += 16) {
    const int j = jb + 4 * wave_id() + (lane >> 4);
    double z[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int i = s + 16 * t;
      z[t] = (i < p && j < nev) ? Z[i * ldz + j] : 0.0;
    }
    double v[NT], b = 0.0;
    auto load = [&](int k) {
      b = beta[k];  // 0 for H_k = I
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int i = s + 16 * t;
        if (PACK) v[t] = (i > k && i < p) ? vref[ref_off(p, k) - (k + 1) + i] : 0.0;
        else v[t] = vref[64 * k + i];
      }
    };
    if (p >= 2) load(p - 2);
    for (int k = p - 2; k >= 0; --k) {
      double vk[NT], dot = 0.0;
      const double nb = -b;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        vk[t] = v[t];
        dot = fma(vk[t], z[t], dot);
      }
      if (k > 0) load(k - 1);
      const double c = nb * row_sum(dot);
#pragma unroll
      for (int t = 0; t < NT; ++t) z[t] = fma(c, vk[t], z[t]);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int i = s + 16 * t;
      if (i < p && j < nev) Z[i * ldz + j] = z[t];
    }
  }
  __syncthreads();
}

// The whole path (1-5) on a (device, p x p) scaled by ds (LDS) from both
// sides; base: LDS laid out by tri_layout(p, nev), whose ev and Z receive the
// result.  Every thread of a kEigThreads workgroup calls it; the return value
// is uniform.
__device__ __forceinline__ bool blk_tri_eigh(const double* __restrict__ a, int p, int nev, const double* ds, double* base,
                             const TriLayout& L) {
  double* d = base + L.d;
  double* e = base + L.e;
  double* beta = base + L.beta;
  double* vref = base + L.vref;
  double* ev = base + L.ev;
  double* Z = base + L.Z;
  dd2* de = reinterpret_cast<dd2*>(base + L.de);
  const int ldz = L.ldz;
  const int lane = threadIdx.x & 63;
  if (p <= 48) reg_tridiag<1, 12>(a, p, ds, d, e, beta, vref, base + L.lu);
  else if (p <= 64) reg_tridiag<1, 16>(a, p, ds, d, e, beta, vref, base + L.lu);
  else reg_tridiag<2, 24>(a, p, ds, d, e, beta, vref, base + L.lu);
  // Gershgorin interval and ||T||, by every wave
  double gl = -INFINITY, gu = -INFINITY;  // (gl holds -min)
  bool bad = false;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h;
    if (i < p) {
      const double r = ((i > 0) ? fabs(e[i - 1]) : 0.0) + ((i + 1 < p) ? fabs(e[i]) : 0.0);
      gl = fmax(gl, r - d[i]);
      gu = fmax(gu, d[i] + r);
      bad |= !(fabs(d[i]) + r < INFINITY);
    }
  }
  if (__ballot(bad) != 0) return false;
  gl = -wave_max(gl);
  gu = wave_max(gu);
  double tnorm = fmax(fabs(gl), fabs(gu));
  if (tnorm == 0.0) {  // the zero matrix
    for (int idx = threadIdx.x; idx < p * nev; idx += kEigThreads) {
      const int i = idx / nev, j = idx - i * nev;
      Z[i * ldz + j] = (i == j) ? 1.0 : 0.0;
    }
    for (int j = threadIdx.x; j < nev; j += kEigThreads) ev[j] = 0.0;
    __syncthreads();
    return true;
  }
  // T scaled by a power of two to ||T|| in [1, 2)
  const int ex = 1 - __builtin_amdgcn_frexp_exp(tnorm);
  tnorm = __builtin_amdgcn_ldexp(tnorm, ex);
  gl = __builtin_amdgcn_ldexp(gl, ex);
  gu = __builtin_amdgcn_ldexp(gu, ex);
  const double tol = kEps * tnorm;
  const double widen = 2.1 * (kEps * tnorm * p);
  gl -= widen;
  gu += widen;
  const int p8 = (p + 7) & ~7;
  __syncthreads();  // the bounds are read
  {
    const int i = threadIdx.x;
    double di = 0.0, ei = 0.0, em = 0.0;
    if (i < p) {
      di = __builtin_amdgcn_ldexp(d[i], ex);
      ei = (i + 1 < p) ? __builtin_amdgcn_ldexp(e[i], ex) : 0.0;
      em = (i > 0) ? __builtin_amdgcn_ldexp(e[i - 1], ex) : 0.0;
    }
    __syncthreads();
    if (i < p) d[i] = di;
    if (i <= p8) e[i] = ei;
    // past the end: |d - x| > 1 with the sign of + and no coupling
    if (i < p + 16) de[i] = (i < p) ? dd2{di, fmax(em * em, 0x1.0p-120)} : dd2{4.0, 0x1.0p-120};
  }
  // start vectors
  for (int idx = threadIdx.x; idx < p8 * nev; idx += kEigThreads) {
    const int i = idx / nev, j = idx - i * nev;
    if (i >= p) {
      Z[i * ldz + j] = 0.0;
      continue;
    }
    const uint64_t z = sm64(kZeroColumnSeed ^ (0x5EEDull << 32) ^ ((uint64_t)j * (uint64_t)p + (uint64_t)i));
    Z[i * ldz + j] = (double)(z >> 11) * 0x1.0p-52 - 1.0;
  }
  __syncthreads();
  blk_multisection(de, p, nev, gl, gu, tnorm, ev);
  __syncthreads();
  // two solves with a Cholesky-QR between them (block inverse iteration;
  // with several batches the LU is rebuilt for the second solve), the
  // back-transformation, then Cholesky-QR twice.  One pass leaves the vectors
  // orthonormal to a few units of rounding when the Gram is well conditioned,
  // yet the second pass is kept: the P coefficients are the small differences
  // u_x - E, and dropping it whenever the columns' cosines were below 1e-3
  // doubled the iterations of a dense generalized solve (n = 2000, 4 pairs:
  // 51 against 25, the lowest pair lagging).
  const int nb = L.nb;
  double* lu = base + L.lu;
  uint64_t sw0 = 0, sw1 = 0;
  for (int stage = 0; stage < 3; ++stage) {
    if (stage < 2) {
      for (int j0 = 0; j0 < nev; j0 += nb) {
        const int t = threadIdx.x, j = j0 + t;
        if (t < nb && j < nev) {
          double *u0 = lu + t, *u1 = u0 + p8 * nb, *lm = u1 + p8 * nb;
          if (stage == 0 || nb < nev) tri_invit_solve<true>(d, e, p, ev[j], tol, Z, ldz, j, u0, u1, lm, nb, sw0, sw1);
          else tri_invit_solve<false>(d, e, p, ev[j], tol, Z, ldz, j, u0, u1, lm, nb, sw0, sw1);
        }
        __syncthreads();
      }
    }
    if (stage == 1) {
      if (p <= 48) blk_backtransform<3, false>(Z, ldz, p, nev, vref, beta);
      else if (p <= 64) blk_backtransform<4, false>(Z, ldz, p, nev, vref, beta);
      else blk_backtransform<6, true>(Z, ldz, p, nev, vref, beta);
      for (int j = threadIdx.x; j < nev; j += kEigThreads) ev[j] = __builtin_amdgcn_ldexp(ev[j], -ex);
    }
    if (!blk_cholqr(Z, ldz, p, nev, base + L.orth)) return false;
  }
  return true;
}

__global__ __launch_bounds__(kEigThreads) void k_small_eigh(const double* __restrict__ a, int p,
                                                            double* __restrict__ evals,
                                                            double* __restrict__ evecs, int* sweeps) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  __shared__ JacobiLds J;
  __shared__ double ds[kMaxP];
  for (int i = threadIdx.x; i < p; i += kEigThreads) ds[i] = 1.0;
  __syncthreads();
  const TriLayout T = tri_layout(p, p);
  if (blk_tri_eigh(a, p, p, ds, smem, T)) {
    for (int idx = threadIdx.x; idx < p * p; idx += kEigThreads) {
      const int i = idx / p, j = idx - i * p;
      const double sg = (smem[T.Z + j * T.ldz + j] < 0.0) ? -1.0 : 1.0;
      evecs[i * p + j] = sg * smem[T.Z + i * T.ldz + j];
    }
    for (int j = threadIdx.x; j < p; j += kEigThreads) evals[j] = smem[T.ev + j];
    if (threadIdx.x == 0 && sweeps != nullptr) *sweeps = 0;
    return;
  }
  __syncthreads();
  const int ld = p + 1;
  double* A = smem;
  double* V = smem + p * ld;
  load_sym(a, p, ds, A, ld);
  const int sw = blk_jacobi<kEigThreads>(A, ld, V, ld, p, J.cs, J.pr, J.flags, J.scratch);
  blk_sort_evals(A, ld, p, J.perm);
  for (int idx = threadIdx.x; idx < p * p; idx += kEigThreads) {
    const int i = idx / p, j = idx - i * p;
    const double sg = (V[j * ld + J.perm[j]] < 0.0) ? -1.0 : 1.0;
    evecs[i * p + j] = sg * V[i * ld + J.perm[j]];
  }
  for (int j = threadIdx.x; j < p; j += kEigThreads) evals[j] = A[J.perm[j] * ld + J.perm[j]];
  if (threadIdx.x == 0 && sweeps != nullptr) *sweeps = sw;
}

hipError_t small_eigh(const double* a, int p, double* evals, double* evecs, int* sweeps,
                      hipStream_t s) {
  if (p < 1 || p > kMaxP) return hipErrorInvalidValue;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)k_small_eigh, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kEigLdsBytes);
    (void)hipGetLastError();
    attr = true;
  }
  hipLaunchKernelGGL(k_small_eigh, dim3(1), dim3(kEigThreads), kEigLdsBytes, s, a, p, evals, evecs, sweeps);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// SVQB (Stathopoulos-Wu) coefficient for an n x n overlap M: X <- X U S^-1/2,
// eigenvalues clamped below eps * max.  Writes the n x n coefficient to Cf.
// Uses Ws (2 * n * (n+1) doubles) as Jacobi workspace.
template <int NT>
__device__ __forceinline__ bool blk_svqb_coef(const double* M, int ldm, int n, double* Cf, int ldc, double* Ws,
                              double* cs, int* pr, int* flag, int* perm, double* scratch) {
  const int ld = n + 1;
  double* A = Ws;
  double* U = Ws + n * ld;
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
    const int i = idx / n, j = idx - i * n;
    A[i * ld + j] = M[i * ldm + j];
  }
  __syncthreads();
  blk_jacobi<NT>(A, ld, U, ld, n, cs, pr, flag, scratch);
  double smax = 0.0;
  for (int i = 0; i < n; ++i) smax = fmax(smax, A[i * ld + i]);
  if (!(smax > 0.0)) return false;
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
    const int i = idx / n, j = idx - i * n;
    const double sj = fmax(A[j * ld + j], kEps * smax);
    Cf[i * ldc + j] = U[i * ld + j] / sqrt(sj);
  }
  __syncthreads();
  return true;
}

// ---------------------------------------------------------------------------
// Rayleigh-Ritz coefficients (Alg. 1): eig of sym(a); u_x = lowest m
// eigenvectors; optionally u_p = ortho(u_x[:, a0:m] - E[:, a0:m]; u_x) in R^p
// by Alg. 3 / Alg. 2 (the same readings as on n-vectors).

// Rayleigh-Ritz coefficients (see small_rr in internal.h).  JAC: the Jacobi
// eigensolver (LOBPCG_OPT_RR_JACOBI), 1024 threads; else the tridiagonal
// path on kEigThreads, with Jacobi where that breaks down.
template <bool JAC>
__global__ __launch_bounds__(JAC ? 1024 : kEigThreads) void k_small_rr(
    const double* __restrict__ a, int p, int m, int a0, int want_up, double tau,
    const OrthoState* __restrict__ pend, int woff, double* __restrict__ theta_all,
    double* __restrict__ U, int* __restrict__ info) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  __shared__ JacobiLds J;
  __shared__ double ds[kMaxP];  // column scaling of V that is still pending
  __shared__ double sg[kMaxP];
  __shared__ ShiftCount cnt;
  __shared__ int zeros;
  __shared__ int stalled, passes, grams, updates;
  if (threadIdx.x == 0) {
    cnt.factorizations = cnt.failed = cnt.shifted = cnt.svqb = 0;
    zeros = stalled = passes = grams = updates = 0;
  }
  {
    const bool scaled = (pend != nullptr) && pend->pending_scale;
    const int nws = scaled ? pend->nw : 0;
    for (int i = threadIdx.x; i < p; i += blockDim.x)
      ds[i] = (i >= woff && i < woff + nws) ? pend->dscale[i - woff] : 1.0;
  }
  __syncthreads();
  int sw = 0;
  // sorted eigenvectors u_x (first m columns), stride ldu, and the LDS after them
  double *Us, *work;
  int ldu;
  bool tri = false;
  if constexpr (!JAC) {
    const TriLayout T = tri_layout(p, m);
    tri = blk_tri_eigh(a, p, m, ds, smem, T);
    if (tri) {
      Us = smem + T.Z;
      ldu = T.ldz;
      work = smem + T.work;
      for (int j = threadIdx.x; j < m; j += blockDim.x) {
        theta_all[j] = smem[T.ev + j];
        // orientation: u[j][j] >= 0, so that u_x - E is the small update X_new - X_old
        sg[j] = (Us[j * ldu + j] < 0.0) ? -1.0 : 1.0;
      }
      __syncthreads();
      for (int idx = threadIdx.x; idx < p * m; idx += blockDim.x) {
        const int i = idx / m, j = idx - i * m;
        Us[i * ldu + j] *= sg[j];
      }
      __syncthreads();
    }
  }
  if (!tri) {
    const int ld = p + 1;
    double* V = smem + p * ld;
    Us = smem;
    ldu = ld;
    work = V;
    __syncthreads();
    load_sym(a, p, ds, Us, ld);
    sw = blk_jacobi<JAC ? 1024 : kEigThreads>(Us, ld, V, ld, p, J.cs, J.pr, J.flags, J.scratch);
    blk_sort_evals(Us, ld, p, J.perm);
    for (int j = threadIdx.x; j < m; j += blockDim.x) theta_all[j] = Us[J.perm[j] * ld + J.perm[j]];
    __syncthreads();
    for (int idx = threadIdx.x; idx < p * p; idx += blockDim.x) {
      const int i = idx / p, j = idx - i * p;
      const double s = (V[j * ld + J.perm[j]] < 0.0) ? -1.0 : 1.0;
      Us[i * ld + j] = s * V[i * ld + J.perm[j]];
    }
    __syncthreads();
  }
  const int na = want_up ? (m - a0) : 0;
  const int q = m + na;
  // 16 lanes to a row of the small matrices from here on
  const int row0 = threadIdx.x >> 4, col0 = threadIdx.x & 15, rstep = blockDim.x >> 4;
  // u_x (row scaling for a pending W scaling is applied when U is written)
  for (int i = row0; i < p; i += rstep)
    for (int j = col0; j < m; j += 16) U[i * q + j] = ds[i] * Us[i * ldu + j];
  int bad = 0;
  if (na > 0) {
    // X (p x na), C (m x na), M and its factor (na x na), SVQB workspace;
    // odd strides, so that a column's entries lie in different banks
    const int ldx = na | 1;
    double* X = work;
    double* C = X + p * ldx;
    double* M = C + m * ldx;
    double* Lc = M + na * ldx;
    double* Ws = Lc + na * ldx;  // max(2 na (na + 1), p na, one transpose per wave)
    // u~_p = u_x[:, a0:m] - E[:, a0:m]
    for (int i = row0; i < p; i += rstep)
      for (int j = col0; j < na; j += 16) X[i * ldx + j] = Us[i * ldu + a0 + j] - ((i == a0 + j) ? 1.0 : 0.0);
    __syncthreads();
    blk_normalize(X, ldx, p, na, &zeros);
    blk_gemm_tn(Us, ldu, X, ldx, p, m, na, C, ldx);  // C = u_x^T X
    for (int pass = 0; pass < 4; ++pass) {
      if (threadIdx.x == 0) passes++;
      blk_sub_mm(X, ldx, Us, ldu, C, ldx, p, m, na);
      // ortho(X): normalise, then Gram / check / shifted Cholesky / X L^-T
      blk_normalize(X, ldx, p, na, &zeros);
      for (int it = 0; it < 6; ++it) {
        if (threadIdx.x == 0) grams++;
        bool fact;
        if (!JAC && na <= 16) {
          // every wave for itself (the same bits), M and its factor in registers
          double g[16], f[16], inv[16];
          gram16_rows(X, ldx, p, na, Ws + wave_id() * kTrans, g);
          double dev = 0.0, diag = 0.0;
#pragma unroll
          for (int c = 0; c < 16; ++c) {
            dev = fmax(dev, fabs(g[c] - (col0 == c ? 1.0 : 0.0)));
            if (col0 == c) diag = g[c];
            f[c] = g[c];
          }
          dev = row_max(dev);
          if (__builtin_amdgcn_readfirstlane(dev <= tau)) break;
          if (it == 5) {
            if (threadIdx.x == 0) stalled++;
            break;
          }
          // plain Cholesky, then shifts (as blk_shifted_chol)
          if (threadIdx.x == 0) cnt.factorizations++;
          fact = chol16_rows(f, na, inv);
          if (!fact) {
            if (threadIdx.x == 0) cnt.failed++;
            const double normx = sqrt(fmax(row_sum(col0 < na ? diag : 0.0), 0.0));
            double alpha = kShiftAlpha0;
            for (int t = 0; t < kShiftRetries && !fact; ++t) {
#pragma unroll
              for (int c = 0; c < 16; ++c) f[c] = g[c] + (col0 == c ? alpha * kEps * normx : 0.0);
              fact = chol16_rows(f, na, inv);
              if (threadIdx.x == 0) {
                cnt.factorizations++;
                if (fact) cnt.shifted++;
                else cnt.failed++;
              }
              alpha *= kShiftGrowth;
            }
          }
          __syncthreads();  // every wave has read X
          if (fact) {
            trsm16_rows(X, ldx, p, na, f, inv);
          } else if (threadIdx.x < 16 && col0 < na) {
#pragma unroll
            for (int c = 0; c < 16; ++c)
              if (c < na) M[col0 * ldx + c] = g[c];
          }
          __syncthreads();
        } else {
          blk_gemm_tn(X, ldx, X, ldx, p, na, na, M, ldx);
          double dev = 0.0;
          for (int i = row0; i < na; i += rstep)
            for (int j = col0; j < na; j += 16)
              dev = fmax(dev, fabs(0.5 * (M[i * ldx + j] + M[j * ldx + i]) - (i == j ? 1.0 : 0.0)));
          dev = blk_reduce_max(dev, J.scratch);
          if (dev <= tau) break;
          if (it == 5) {
            if (threadIdx.x == 0) stalled++;
            break;
          }
          // (both halves of M are read: the pair (i, j), (j, i) by one thread)
          for (int i = row0; i < na; i += rstep)
            for (int j = col0; j < i; j += 16) {
              const double v = 0.5 * (M[i * ldx + j] + M[j * ldx + i]);
              M[i * ldx + j] = v;
              M[j * ldx + i] = v;
            }
          __syncthreads();
          fact = blk_shifted_chol(M, ldx, na, Lc, ldx, J.flags, &cnt);
          if (fact) blk_trsm_rt(X, ldx, p, na, Lc, ldx);
        }
        if (!fact) {
          if (threadIdx.x == 0) cnt.svqb++;
          if (!blk_svqb_coef<JAC ? 1024 : kEigThreads>(M, ldx, na, Lc, ldx, Ws, J.cs, J.pr, J.flags, J.perm, J.scratch)) {
            bad = 1;
            break;
          }
          // X <- X Cf (Cf in Lc), through the Ws area as a copy of X
          for (int idx = threadIdx.x; idx < p * na; idx += blockDim.x) Ws[idx] = X[idx / na * ldx + idx % na];
          __syncthreads();
          for (int idx = threadIdx.x; idx < p * na; idx += blockDim.x) {
            const int r = idx / na, j = idx - r * na;
            double acc = 0.0;
            for (int k = 0; k < na; ++k) acc += Ws[r * na + k] * Lc[k * ldx + j];
            X[r * ldx + j] = acc;
          }
          __syncthreads();
        }
        if (threadIdx.x == 0) updates++;
      }
      if (bad) break;
      blk_gemm_tn(Us, ldu, X, ldx, p, m, na, C, ldx);
      double cm = 0.0;
      for (int i = row0; i < m; i += rstep)
        for (int j = col0; j < na; j += 16) cm = fmax(cm, fabs(C[i * ldx + j]));
      cm = blk_reduce_max(cm, J.scratch);
      if (cm <= tau) break;
      if (pass == 3 && threadIdx.x == 0) stalled++;
    }
    for (int i = row0; i < p; i += rstep)
      for (int j = col0; j < na; j += 16) U[i * q + m + j] = ds[i] * X[i * ldx + j];
  }
  if (threadIdx.x == 0) {
    info[0] = sw;
    info[1] = bad;
    info[2] = grams;
    info[3] = cnt.factorizations;
    info[4] = cnt.failed;
    info[5] = cnt.shifted;
    info[6] = updates;
    info[7] = passes;
    info[8] = stalled;
    info[9] = cnt.svqb;
    info[10] = zeros;
    info[11] = (tri || JAC) ? 0 : 1;  // Jacobi fallback of the eigensolve
  }
}

// u~_p's arrays (k_small_rr's carve-up) behind u_x: p x (p + 1) of it after
// Jacobi, less on the tridiagonal path
static_assert(kMaxP * (kMaxP + 1) + kMaxP * (kMaxBlock | 1) + 3 * kMaxBlock * (kMaxBlock | 1) + kMaxP * kMaxBlock <=
                      kEigLdsBytes / 8 &&
                  kMaxP >= 2 * (kMaxBlock + 1) - 1,
              "LDS of the largest Rayleigh-Ritz call");

template <bool JAC>
static hipError_t small_rr_launch(const double* a, int p, int m, int a0, int want_up, double tau,
                                  const OrthoState* pend, int woff, double* theta_all, double* U, int* info,
                                  hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    // dynamic + static LDS must stay within the 160 KB of a workgroup
    (void)hipFuncSetAttribute((const void*)k_small_rr<JAC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kEigLdsBytes);
    (void)hipGetLastError();
    attr = true;
  }
  hipLaunchKernelGGL(k_small_rr<JAC>, dim3(1), dim3(JAC ? 1024 : kEigThreads), kEigLdsBytes, s, a, p, m, a0,
                     want_up, tau, pend, woff, theta_all, U, info);
  return hipGetLastError();
}

hipError_t small_rr(const double* a, int p, int m, int a0, int want_up, double tau,
                    const OrthoState* pend, int woff, double* theta_all, double* U, int* info,
                    int jacobi, hipStream_t s) {
  if (p < 1 || p > kMaxP || m < 1 || m > p || m > kMaxBlock || a0 < 0 || a0 > m) return hipErrorInvalidValue;
  return jacobi ? small_rr_launch<true>(a, p, m, a0, want_up, tau, pend, woff, theta_all, U, info, s)
                : small_rr_launch<false>(a, p, m, a0, want_up, tau, pend, woff, theta_all, U, info, s);
}

// ---------------------------------------------------------------------------
// standalone shifted Cholesky (p <= 64)

__global__ __launch_bounds__(256) void k_small_chol(const double* __restrict__ M, int p,
                                                    double* __restrict__ Lout, int* info) {
  __shared__ double Ms[64 * 65];
  __shared__ double Ls[64 * 65];
  __shared__ int flag;
  __shared__ ShiftCount cnt;
  if (threadIdx.x == 0) cnt.factorizations = cnt.failed = cnt.shifted = cnt.svqb = 0;
  for (int idx = threadIdx.x; idx < p * p; idx += blockDim.x) {
    const int i = idx / p, j = idx - i * p;
    Ms[i * 65 + j] = 0.5 * (M[i * p + j] + M[j * p + i]);
  }
  __syncthreads();
  const bool ok = blk_shifted_chol<false>(Ms, 65, p, Ls, 65, &flag, &cnt);
  for (int idx = threadIdx.x; idx < p * p; idx += blockDim.x) {
    const int i = idx / p, j = idx - i * p;
    Lout[idx] = ok ? Ls[i * 65 + j] : 0.0;
  }
  if (threadIdx.x == 0) {
    info[0] = ok ? 0 : 1;
    info[1] = cnt.factorizations;
    info[2] = cnt.failed;
    info[3] = cnt.shifted;
  }
}

hipError_t small_cholesky(const double* M, int p, double* L, int* info, hipStream_t s) {
  if (p < 1 || p > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_small_chol, dim3(1), dim3(256), 0, s, M, p, L, info);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// ortho(W; Y) controller.  G = [Y W]^T W, (ny + nw) x nw: rows [0, ny) are
// C = Y^T W, rows [ny, ny+nw) are M = W^T W.  The coefficient written to
// `coef` ((ny+nw) x nw) is applied by the streaming kernel as
// W <- [Y W] coef, after which G is recomputed and this kernel runs again.
//
// Phases (reading of Alg. 3 as a do-while around Alg. 2, both with column
// normalisation first):
//   START  raw W~: normalise (D0) and project: coef = [-C D0; D0]
//          (no Y: behave as BEGIN)
//   BEGIN  start of ortho(X): D = diag(M)^-1/2, M' = D M D;
//          ||M' - I|| <= tau -> ortho done on X = W D: Alg. 3 check on C D;
//          else shifted Cholesky M' = L L^T, coef = [0; D L^-T] -> LOOP
//   LOOP   ||M - I|| <= tau (or pass cap) -> Alg. 3 check on C;
//          else shifted Cholesky, coef = [0; L^-T]
//   Alg. 3 check: ||C|| <= tau (or no Y) -> finished; else project
//          coef = [-C; I] (scaled by the pending D) -> BEGIN
//   FINAL  a pending diagonal scaling was applied: finished.

enum { kPhFinal = 5, kPhYCheck = 6 };

// Bound on ||L^-1||_2 for the n x n lower factor L (stride ldl) with its
// inverse Li (stride ldi): 1 / (1 - e) when e = ||I - L||_F < 1/2 (Neumann
// series), else ||Li||_F.  *e_out receives e.  Every thread gets the result.
__device__ double blk_inv_bound(const double* L, int ldl, const double* Li, int ldi, int n,
                                double* e_out, double* scratch) {
  double se = 0.0, si = 0.0;
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
    const int i = idx / n, j = idx - i * n;
    if (j > i) continue;
    const double d = (i == j ? 1.0 : 0.0) - L[i * ldl + j];
    se += d * d;
    const double v = Li[i * ldi + j];
    si += v * v;
  }
  se = blk_reduce_sum_ordered(se, scratch);
  si = blk_reduce_sum_ordered(si, scratch);
  const double e = sqrt(se);
  *e_out = e;
  return (e < 0.5) ? 1.0 / (1.0 - e) : sqrt(si);
}

__global__ __launch_bounds__(1024) void k_ortho_ctl(const double* __restrict__ G,
                                                   OrthoState* __restrict__ gst,
                                                   double* __restrict__ coef) {
  __shared__ OrthoState st;
  __shared__ double Gs[kMaxP * kMaxBlock];
  __shared__ double Ms[kMaxBlock * (kMaxBlock + 1)];
  __shared__ double Ls[kMaxBlock * (kMaxBlock + 1)];
  __shared__ double Li[kMaxBlock * (kMaxBlock + 1)];
  __shared__ double Ws[2 * kMaxBlock * (kMaxBlock + 1)];
  __shared__ double D[kMaxBlock];
  __shared__ double cs[3 * 64];
  __shared__ int pr[2 * 64];
  __shared__ int perm[64];
  __shared__ double scratch[16];
  __shared__ int flag, nonfinite, zero_mask;
  __shared__ ShiftCount cnt;
  if (threadIdx.x == 0) {
    st = *gst;
    nonfinite = 0;
    zero_mask = 0;
    cnt.factorizations = cnt.failed = cnt.shifted = cnt.svqb = 0;
  }
  __syncthreads();
  if (st.done) return;
  const int ny = st.ny, nw = st.nw, nr = ny + nw;
  const int ldm = kMaxBlock + 1;
  for (int idx = threadIdx.x; idx < nr * nw; idx += blockDim.x) {
    const double v = G[idx];
    Gs[idx] = v;
    if (!isfinite(v)) nonfinite = 1;
  }
  __syncthreads();
  if (st.state == kPhFinal) {
    if (threadIdx.x == 0) {
      st.done = 1;
      st.skip_sum = 1;
      st.state = kPhDone;
      *gst = st;
    }
    return;
  }
  if (threadIdx.x == 0) st.grams++;  // (a no-overlap apply only precedes kPhFinal)
  if (nonfinite) {
    if (threadIdx.x == 0) {
      st.error = kOrthoErrNonfinite;
      st.done = 1;
      st.skip_sum = 1;
      *gst = st;
    }
    return;
  }
  // symmetrised M
  for (int idx = threadIdx.x; idx < nw * nw; idx += blockDim.x) {
    const int i = idx / nw, j = idx - i * nw;
    Ms[i * ldm + j] = 0.5 * (Gs[(ny + i) * nw + j] + Gs[(ny + j) * nw + i]);
  }
  __syncthreads();
  int phase = st.state;
  if (phase == kPhStart && ny == 0) phase = kPhBegin;

  // helper lambdas are avoided: explicit code per phase
  bool check_outer = false;
  bool have_scale = false;  // D pending (BEGIN passed its check)
  bool capped = false;
  double growth = st.growth;  // amplification of errors by the current Alg. 2 call
  if (phase == kPhStart || phase == kPhBegin) {
    for (int j = threadIdx.x; j < nw; j += blockDim.x) {
      const double d = Ms[j * ldm + j];
      if (d == 0.0) atomicOr(&zero_mask, 1 << j);
      D[j] = (d > 0.0) ? 1.0 / sqrt(d) : 0.0;
    }
    __syncthreads();
    if (zero_mask) {
      if (threadIdx.x == 0) {
        st.error = kOrthoErrZero;
        st.zero_mask = zero_mask;
        st.done = 1;
        st.skip_sum = 1;
        *gst = st;
      }
      return;
    }
  }
  if (phase == kPhStart) {
    // normalise + first projection (Alg. 3, first pass)
    for (int idx = threadIdx.x; idx < nr * nw; idx += blockDim.x) {
      const int i = idx / nw, j = idx - i * nw;
      coef[idx] = (i < ny) ? -Gs[i * nw + j] * D[j] : ((i - ny == j) ? D[j] : 0.0);
    }
    if (threadIdx.x == 0) {
      st.passes++;
      st.outer = 1;
      st.w_only = 0;
      st.no_gram = 0;
      st.skip_sum = 0;
      st.state = kPhBegin;
      *gst = st;
    }
    return;
  }
  if (phase == kPhBegin) {
    // M' = D M D, Alg. 2 check on the normalised X; the normalisation is
    // the first factor of this Alg. 2 call's growth
    double dmax = 0.0;
    for (int j = threadIdx.x; j < nw; j += blockDim.x) dmax = fmax(dmax, D[j]);
    growth = blk_reduce_max(dmax, scratch);
    for (int idx = threadIdx.x; idx < nw * nw; idx += blockDim.x) {
      const int i = idx / nw, j = idx - i * nw;
      Ms[i * ldm + j] *= D[i] * D[j];
    }
    if (threadIdx.x == 0) st.inner = 1;
    __syncthreads();
  } else if (phase == kPhLoop || phase == kPhYCheck) {
    if (threadIdx.x == 0 && phase == kPhLoop) st.inner++;
    for (int j = threadIdx.x; j < nw; j += blockDim.x) D[j] = 1.0;
    __syncthreads();
  }
  if (phase == kPhYCheck) {
    // a cheap exit ended Alg. 2 with the last update; only the Alg. 3
    // check of Y^T W (in the overlap that update formed) remains
    check_outer = true;
  } else {
  double dev = 0.0;
  for (int idx = threadIdx.x; idx < nw * nw; idx += blockDim.x) {
    const int i = idx / nw, j = idx - i * nw;
    dev = fmax(dev, fabs(Ms[i * ldm + j] - (i == j ? 1.0 : 0.0)));
  }
  dev = blk_reduce_max(dev, scratch);
  const bool ortho_ok = dev <= st.tau;
  capped = !ortho_ok && st.inner >= st.max_inner;
  if (ortho_ok || capped) {
    if (capped && threadIdx.x == 0) st.stalled++;
    check_outer = true;
    have_scale = (phase == kPhBegin);
  } else {
    // shifted Cholesky of M (= M' in BEGIN)
    const bool ok = blk_shifted_chol(Ms, ldm, nw, Ls, ldm, &flag, &cnt, st.shift_retries);
    if (ok) {
      blk_tri_inv(Ls, ldm, nw, Li, ldm);
      // coef W part: D L^-T, i.e. coef[ny+i][j] = D_i Linv[j][i]
      for (int idx = threadIdx.x; idx < nr * nw; idx += blockDim.x) {
        const int i = idx / nw, j = idx - i * nw;
        coef[idx] = (i < ny) ? 0.0 : D[i - ny] * Li[j * ldm + (i - ny)];
      }
      // cheap exits: e = ||I - L||_F bounds kappa(L) <= (1 + e) / (1 - e)
      // and ||L^-1||; when the pass provably reached tau the overlap of the
      // new W is not formed (Alg. 2), and when the growth of the whole
      // Alg. 2 call also keeps Y^T W below tau, neither is Y^T W (Alg. 3)
      double e = 1.0;
      const double b = blk_inv_bound(Ls, ldm, Li, ldm, nw, &e, scratch);
      growth *= b;
      const double kap = (1.0 + e) / (1.0 - e);
      const bool exit2 = st.cheap_exit && cnt.shifted == 0 && e < 0.5 &&
                         st.cexit * kap * kap <= st.tau;
      const bool exit3 = exit2 && (ny == 0 || st.cexit * growth <= st.tau);
      if (threadIdx.x == 0) {
        st.factorizations += cnt.factorizations;
        st.failed += cnt.failed;
        st.shifted += cnt.shifted;
        st.svqb += cnt.svqb;
        st.updates++;
        st.w_only = 1;
        st.growth = growth;
        if (exit2) st.cheap_exits += (exit3 && ny > 0) ? 2 : 1;
        st.no_gram = exit3 ? 1 : 0;
        st.skip_sum = st.no_gram;
        st.state = exit3 ? kPhFinal : (exit2 ? kPhYCheck : kPhLoop);
        *gst = st;
      }
      return;
    } else {
      if (threadIdx.x == 0) cnt.svqb++;
      const bool sv = blk_svqb_coef<1024>(Ms, ldm, nw, Li, ldm, Ws, cs, pr, &flag, perm, scratch);
      if (!sv) {
        if (threadIdx.x == 0) {
          st.error = kOrthoErrFailed;
          st.done = 1;
          st.skip_sum = 1;
          st.factorizations += cnt.factorizations;
          st.failed += cnt.failed;
          *gst = st;
        }
        return;
      }
      for (int idx = threadIdx.x; idx < nr * nw; idx += blockDim.x) {
        const int i = idx / nw, j = idx - i * nw;
        coef[idx] = (i < ny) ? 0.0 : D[i - ny] * Li[(i - ny) * ldm + j];
      }
    }
    if (threadIdx.x == 0) {
      st.factorizations += cnt.factorizations;
      st.failed += cnt.failed;
      st.shifted += cnt.shifted;
      st.svqb += cnt.svqb;
      st.updates++;
      st.w_only = 1;
      st.growth = INFINITY;  // SVQB: no growth bound, no cheap exit
      st.no_gram = 0;
      st.skip_sum = 0;
      st.state = kPhLoop;
      *gst = st;
    }
    return;
  }
  }
  // Alg. 3: the growth of the finished Alg. 2 call may already bound Y^T W
  // below tau (cheap exit); else check C D (D = 1 unless BEGIN's
  // normalisation is pending)
  const bool grow_ok = st.cheap_exit && ny > 0 && !capped && phase != kPhYCheck &&
                       st.cexit * growth <= st.tau;
  double cm = 0.0;
  for (int idx = threadIdx.x; idx < ny * nw; idx += blockDim.x) {
    const int j = idx % nw;
    cm = fmax(cm, fabs(Gs[idx] * D[j]));
  }
  cm = blk_reduce_max(cm, scratch);
  if (grow_ok && threadIdx.x == 0) st.cheap_exits++;
  const bool y_ok = (ny == 0) || grow_ok || (cm <= st.tau);
  if (y_ok || st.outer >= st.max_outer) {
    if (!y_ok && threadIdx.x == 0) st.stalled++;
    if (have_scale && st.fold_scale) {
      // leave the normalisation pending: the caller folds it into the next
      // Rayleigh-Ritz coefficients instead of spending a pass on it
      if (threadIdx.x == 0) {
        for (int j = 0; j < nw; ++j) st.dscale[j] = D[j];
        st.pending_scale = 1;
        st.done = 1;
        st.skip_sum = 1;
        st.state = kPhDone;
        *gst = st;
      }
    } else if (have_scale) {
      // apply the pending normalisation, then finish
      for (int idx = threadIdx.x; idx < nr * nw; idx += blockDim.x) {
        const int i = idx / nw, j = idx - i * nw;
        coef[idx] = (i < ny) ? 0.0 : ((i - ny == j) ? D[j] : 0.0);
      }
      if (threadIdx.x == 0) {
        st.w_only = 1;
        st.no_gram = 1;  // the next round only finishes
        st.skip_sum = 1;
        st.state = kPhFinal;
        *gst = st;
      }
    } else if (threadIdx.x == 0) {
      st.done = 1;
      st.skip_sum = 1;
      st.state = kPhDone;
      *gst = st;
    }
    return;
  }
  // project again: W <- W D - Y (C D)
  for (int idx = threadIdx.x; idx < nr * nw; idx += blockDim.x) {
    const int i = idx / nw, j = idx - i * nw;
    coef[idx] = (i < ny) ? -Gs[i * nw + j] * D[j] : ((i - ny == j) ? D[j] : 0.0);
  }
  if (threadIdx.x == 0) {
    st.passes++;
    st.outer++;
    st.w_only = 0;
    st.no_gram = 0;
    st.skip_sum = 0;
    st.state = kPhBegin;
    *gst = st;
  }
}

__global__ void k_ortho_init(OrthoState* st, int ny, int nw, double tau, int max_inner,
                             int max_outer, int shift_retries, int fold_scale, double cexit) {
  OrthoState s;
  s.state = kPhStart;
  s.done = 0;
  s.inner = 0;
  s.outer = 0;
  s.w_only = 0;
  s.error = 0;
  s.zero_mask = 0;
  s.grams = s.factorizations = s.failed = s.shifted = s.updates = s.stalled = s.svqb = s.passes = 0;
  s.ny = ny;
  s.nw = nw;
  s.max_inner = max_inner;
  s.max_outer = max_outer;
  s.shift_retries = shift_retries;
  s.fold_scale = fold_scale;
  s.pending_scale = 0;
  s.cheap_exit = cexit > 0.0 ? 1 : 0;
  s.cheap_exits = 0;
  s.no_gram = 0;
  s.skip_sum = 0;
  s.cexit = cexit;
  s.growth = INFINITY;
  s.tau = tau;
  for (int j = 0; j < kMaxBlock; ++j) s.dscale[j] = 1.0;
  *st = s;
}

hipError_t ortho_init(OrthoState* st, int ny, int nw, double tau, int max_inner, int max_outer,
                      int shift_retries, int fold_scale, double cexit, hipStream_t s) {
  if (nw < 1 || nw > kMaxBlock || ny < 0 || ny + nw > kMaxP || shift_retries < 0)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_ortho_init, dim3(1), dim3(1), 0, s, st, ny, nw, tau, max_inner, max_outer,
                     shift_retries, fold_scale, cexit);
  return hipGetLastError();
}

hipError_t ortho_ctl(const double* G, OrthoState* st, double* coef, hipStream_t s) {
  // 1024 threads: the SVQB fallback runs the Jacobi sweep, which assumes them
  hipLaunchKernelGGL(k_ortho_ctl, dim3(1), dim3(1024), 0, s, G, st, coef);
  return hipGetLastError();
}

}  // namespace lobpcg
