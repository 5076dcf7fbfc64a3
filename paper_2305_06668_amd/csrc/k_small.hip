// Small dense fp64 linear algebra of the LOBPCG step, one workgroup each,
// everything resident in LDS (gfx950: 160 KB per workgroup):
//   * the eigensolve of the p x p Rayleigh-Ritz matrix, p <= 96 (Alg. 1,
//     "solve a u = lambda u"; the paper calls LAPACK dsyev, Sec. 3.1);
//   * shifted Cholesky of an overlap matrix (Sec. 3.2: retry with
//     alpha * eps * ||X|| added to the diagonal, alpha = 100, 1000, ...);
//   * the implicit P coefficients u_p = ortho(u_x[:, act] - E[:, act]; u_x)
//     in R^p (Alg. 1 and the "Basis selection" paragraph of Sec. 3.1);
//   * the controller of ortho(W; Y) on n-vectors (Alg. 2 inside Alg. 3): it
//     reads the overlap G = [Y W]^T W of the current W and emits the small
//     coefficient matrix that the streaming kernel applies next.
#include <cstring>

#include "small.h"

namespace lobpcg {

namespace {

constexpr double kShiftAlpha0 = 100.0;
constexpr double kShiftGrowth = 10.0;
constexpr int kShiftRetries = 20;

// L = chol(S + shift I) for the n x n (n <= 16) matrix S in LDS by one wave (all
// 64 lanes), written to L in LDS with zeros above the diagonal.  Lane l keeps
// column c = l & 15, rows r = (l >> 4) + 4 t (t = 0..3), in g[t]; only r >= c is
// read, and rows or columns from n to 15 are those of the identity.
// Right-looking, column by column: the pivot is read from its lane, column k of L
// is formed in its four lanes and handed to the others by lane shuffles, then the
// trailing entries are updated.  Every entry takes the operations of the LDS
// factorization in its order: G[r][k] / l_kk, and G[r][c] - L[r][k] L[c][k] as one
// fused multiply-add.  False (uniform) on a pivot that is not > 0.
__device__ __forceinline__ bool wave_chol16(const double* S, int lds_, int n, double shift, double* L, int ldl) {
  const int l = threadIdx.x & 63, c = l & 15, rb = l >> 4;
  double g[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int r = rb + 4 * t;
    g[t] = (r < n && c < n) ? ((r >= c) ? S[r * lds_ + c] + (r == c ? shift : 0.0) : 0.0)
                            : (r == c ? 1.0 : 0.0);
  }
  bool ok = true;
  for (int k = 0; k < n; ++k) {
    // register k >> 2 of lane k + 16 (k & 3) (a select: no indexed registers)
    const int tk = k >> 2;
    const double gk = (tk == 0) ? g[0] : (tk == 1) ? g[1] : (tk == 2) ? g[2] : g[3];
    const double gkk = readlane_f64(gk, k + 16 * (k & 3));
    if (!(gkk > 0.0)) {
      ok = false;
      break;
    }
    const double lkk = sqrt(gkk);
    if (c == k) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = rb + 4 * t;
        if (r > k) g[t] = g[t] / lkk;
        else if (r == k) g[t] = lkk;
      }
    }
    // lr[t] = L[rb + 4t][k] (lane k + 16 rb, register t); lc[t] from lane
    // k + 16 (c & 3): L[c][k] is its register c >> 2
    double lr[4], lc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      lr[t] = __shfl(g[t], k + 16 * rb);
      lc[t] = __shfl(g[t], k + 16 * (c & 3));
    }
    const int tc = c >> 2;
    const double lck = (tc == 0) ? lc[0] : (tc == 1) ? lc[1] : (tc == 2) ? lc[2] : lc[3];
    if (c > k) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (rb + 4 * t >= c) g[t] = fma(-lr[t], lck, g[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int r = rb + 4 * t;
    if (r < n && c < n) L[r * ldl + c] = (r >= c) ? g[t] : 0.0;
  }
  return ok;
}
// Cholesky of an n x n matrix (n <= N <= 16) in LDS by one wave, each row of 16
// lanes with a copy of its own: lane l holds matrix row l % 16 in g (only the
// lower triangle is read; rows and columns from n to N - 1 are those of the
// identity).  The pivot is handed on by DPP, so a column costs a root, a
// division, a product and an update in sequence (220 cycles; by lane shuffles
// through LDS 1100).  Every entry takes the operations of wave_chol16 in its
// order: G[r][k] / l_kk (KDIV) or G[r][k] * (1 / l_kk), and
// G[r][c] - L[r][k] L[c][k] as one fused multiply-add.  On return g holds L
// and inv the reciprocals of its diagonal (!KDIV).  False, uniform, when a
// pivot is not > 0 (or, CHECKINF, not finite).
template <int N, bool KDIV, bool CHECKINF>
__device__ __forceinline__ bool chol16_rows(const double* G, int ldg, int n, double (&g)[N], double (&inv)[N]) {
  const int r = threadIdx.x & 15;
  const double* Gr = G + min(r, n - 1) * ldg;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const double v = Gr[min(c, n - 1)];
    g[c] = ((r < n) & (c < n) & (r >= c)) ? v : ((r == c) ? 1.0 : 0.0);
  }
  bool bad = false;
  static_for<0, N>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    const double gkk = row_bcast<k>(g[k]);
    bad |= !(gkk > 0.0) | (CHECKINF & !(gkk < INFINITY));
    const double lkk = sqrt(gkk);
    double below;
    if (KDIV) {
      below = g[k] / lkk;
    } else {
      inv[k] = 1.0 / lkk;
      below = g[k] * inv[k];
    }
    g[k] = (r > k) ? below : (r == k) ? lkk : g[k];
    static_for<k + 1, N>([&](auto cc) {
      constexpr int c = decltype(cc)::value;
      const double lck = row_bcast<c>(g[k]);
      g[c] = fma(-g[k], lck, g[c]);  // (r < c: not used)
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  // (or the broadcasts above would be kept, two registers each, for the solves)
#pragma unroll
  for (int c = 0; c < N; ++c) asm("" : "+v"(g[c]));
  return __ballot(bad) == 0;
}
// X (p x n) <- X L^-T for row i of this lane, L in g as chol16_rows leaves it.
// KDIV: z_j = (x_j - sum_{k<j} z_k L_jk) / L_jj, summed in order; else the sum
// runs over even and odd k apart and the reciprocal multiplies it.
template <int N, bool KDIV>
__device__ __forceinline__ void trsm16_rows(double* X, int ldx, int i, int p, int n, const double (&g)[N],
                                            const double (&inv)[N]) {
  double z[N];
  double* Xi = X + min(i, p - 1) * ldx;
#pragma unroll
  for (int j = 0; j < N; ++j) z[j] = Xi[min(j, n - 1)];
  static_for<0, N>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    if (KDIV) {
      double t = z[j];
      static_for<0, j>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        t = fma(-z[k], row_bcast<j>(g[k]), t);
      });
      z[j] = t / row_bcast<j>(g[j]);
    } else {
      double s0 = z[j], s1 = 0.0;
      static_for<0, j>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        const double ljk = row_bcast<j>(g[k]);
        if (k % 2 == 0) s0 = fma(-z[k], ljk, s0);
        else s1 = fma(-z[k], ljk, s1);
      });
      z[j] = (s0 + s1) * inv[j];
    }
    asm volatile("" : "+v"(z[j]));  // (computed here, not where it is stored: the broadcasts would stay)
  });
  if (i < p) {
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (j < n) Xi[j] = z[j];
  }
}
// L = chol(M) and its inverse (both n x n in LDS, zero above the diagonal) by
// one wave: lane j % 16 solves for column j of the inverse in its registers,
// the operations and their order those of blk_tri_inv (the terms above the
// diagonal add zeros).  A root and two divisions per column, one after the
// other: 4.4 us for n = 16 (solving a row beside the next column of the factor
// gains nothing).
template <int N>
__device__ __forceinline__ bool chol_inv16(const double* M, int ldm, int n, double* L, int ldl, double* Li, int ldi) {
  const int r = threadIdx.x & 15;
  double g[N], inv[N];
  if (!chol16_rows<N, true, false>(M, ldm, n, g, inv)) return false;
  double z[N];
  static_for<0, N>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    double t = (r == i) ? 1.0 : 0.0;
    static_for<0, i>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      t = fma(-row_bcast<i>(g[k]), z[k], t);
    });
    z[i] = t / row_bcast<i>(g[i]);
    asm volatile("" : "+v"(z[i]));  // (computed here, not where it is stored: the broadcasts would stay)
  });
  if ((threadIdx.x & 63) < n) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (i < n) {
        L[r * ldl + i] = (i <= r) ? g[i] : 0.0;
        Li[i * ldi + r] = z[i];
      }
  }
  return true;
}
// factor and solve, by the waves that have rows (64 to a wave); the flag (LDS) is 1 on success
template <int N, bool KDIV, bool CHECKINF>
__device__ __forceinline__ void chol_trsm(double* X, int ldx, int p, int n, const double* G, int ldg, int* flag) {
  if (64 * wave_id() < p) {
    double g[N], inv[N];
    const bool ok = chol16_rows<N, KDIV, CHECKINF>(G, ldg, n, g, inv);
    if (ok) trsm16_rows<N, KDIV>(X, ldx, 64 * wave_id() + (threadIdx.x & 63), p, n, g, inv);
    if (threadIdx.x == 0) *flag = ok ? 1 : 0;
  }
}

// ---------------------------------------------------------------------------
// block-wide helpers (every thread of the block calls them)

// ---- small products on the fp64 MFMA 16x16x4 -------------------------------
// Lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator register
// r is row 4 r + l / 16, column l % 16.  An accumulator takes its products one
// after the other, k ascending, each as a fused multiply-add: the bits of the
// scalar loop s = fma(a, b, s).
typedef double d4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ d4 mma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// f(i, j, sum) over the entries of A^T B (A: K x m, B: K x n), a wave per 16 x 16 tile
template <class F>
__device__ __forceinline__ void blk_tiles_tn(const double* A, int lda, const double* B, int ldb, int K, int m, int n,
                                             F&& f) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int tm = (m + 15) >> 4, tn = (n + 15) >> 4;
  for (int t = wave_id(); t < tm * tn; t += blockDim.x >> 6) {
    const int i0 = 16 * (tn == 1 ? t : t / tn), j0 = tn == 1 ? 0 : 16 * (t % tn);
    const bool vi = i0 + r < m, vj = j0 + r < n;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < K; k0 += 16) {
      double av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + 4 * u + g, kc = min(k, K - 1);
        const double x = A[kc * lda + min(i0 + r, m - 1)], y = B[kc * ldb + min(j0 + r, n - 1)];
        av[u] = (vi & (k < K)) ? x : 0.0;
        bv[u] = (vj & (k < K)) ? y : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = mma64(av[u], bv[u], acc);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 4 * q + g;
      if (i < m && vj) f(i, j0 + r, acc[q]);
    }
  }
}
// C (p x q) = A^T B, A: n x p, B: n x q
__device__ __forceinline__ void blk_gemm_tn(const double* A, int lda, const double* B, int ldb, int n, int p,
                            int q, double* C, int ldc) {
  blk_tiles_tn(A, lda, B, ldb, n, p, q, [&](int i, int j, double v) { C[i * ldc + j] = v; });
  __syncthreads();
}

// X (n x q) -= Y (n x p) C (p x q)
__device__ __forceinline__ void blk_sub_mm(double* X, int ldx, const double* Y, int ldy, const double* C, int ldc,
                           int n, int p, int q) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int tm = (n + 15) >> 4, tn = (q + 15) >> 4;
  for (int t = wave_id(); t < tm * tn; t += blockDim.x >> 6) {
    const int i0 = 16 * (tn == 1 ? t : t / tn), j0 = tn == 1 ? 0 : 16 * (t % tn);
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < p; k0 += 16) {
      double av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + 4 * u + g;
        const double x = Y[min(i0 + r, n - 1) * ldy + min(k, p - 1)], y = C[min(k, p - 1) * ldc + min(j0 + r, q - 1)];
        av[u] = ((i0 + r < n) & (k < p)) ? x : 0.0;
        bv[u] = ((j0 + r < q) & (k < p)) ? y : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = mma64(av[u], bv[u], acc);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 4 * u + g;
      if (i < n && j0 + r < q) X[i * ldx + j0 + r] -= acc[u];
    }
  }
  __syncthreads();
}

// scale columns of X (n x q) to unit norm; exact-zero columns are replaced
// by SplitMix64 columns (entry i of column j: splitmix64(seed + j n + i)).
__device__ __forceinline__ void blk_normalize(double* X, int ldx, int n, int q, double* tmp, int* zeros) {
  for (int j = threadIdx.x; j < q; j += blockDim.x) {
    double s = 0.0;
#pragma unroll 16
    for (int r = 0; r < n; ++r) s += X[r * ldx + j] * X[r * ldx + j];
    if (s == 0.0) {
      for (int r = 0; r < n; ++r) {
        const uint64_t z = sm64(kZeroColumnSeed + (uint64_t)j * (uint64_t)n + (uint64_t)r);
        X[r * ldx + j] = (double)(z >> 11) * 0x1.0p-53 - 0.5;
      }
      s = 0.0;
      for (int r = 0; r < n; ++r) s += X[r * ldx + j] * X[r * ldx + j];
      atomicAdd(zeros, 1);
    }
    tmp[j] = sqrt(s);
  }
  __syncthreads();
  for (int j = threadIdx.x & 15; j < q; j += 16)
    for (int r = threadIdx.x >> 4; r < n; r += blockDim.x >> 4) X[r * ldx + j] /= tmp[j];
  __syncthreads();
}

// Cholesky L L^T = M + shift I (lower, n x n); returns true on success.
// Breaks down when a pivot is not > 0 (NaN included), like LAPACK potrf.
// Every thread calls it and M must be complete on entry.  Wave 0 alone
// factors (REG and n <= 16: in registers, in the ortho controller and the
// Rayleigh-Ritz kernel with the Jacobi option; otherwise column by column in
// LDS with wave-level syncs) while the other waves wait at the closing
// barriers: two workgroup barriers per factorization.  Each entry takes the
// same operations in the same order as a column-parallel factorization by the
// whole workgroup.
template <bool REG>
__device__ __forceinline__ bool blk_chol(const double* M, int ldm, int n, double shift, double* L, int ldl,
                         int* flag) {
  if (REG && threadIdx.x < 64 && n <= 16) {
    const bool ok = wave_chol16(M, ldm, n, shift, L, ldl);
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
// ||X||_F = sqrt(trace M), alpha = 100, x10 per retry.  plain = false: the
// caller has tried the plain one, and failed.
template <bool REG>
__device__ __forceinline__ bool blk_shifted_chol(const double* M, int ldm, int n, double* L, int ldl, int* flag,
                                 ShiftCount* c, int retries = kShiftRetries, bool plain = true) {
  if (threadIdx.x == 0) c->factorizations++;
  if (plain && blk_chol<REG>(M, ldm, n, 0.0, L, ldl, flag)) return true;
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

// LDS layout shared by the eig-based kernels
struct EigLds {
  double* A;  // p x (p+1)
  double* V;  // p x (p+1)
  double* cs;
  int* pr;
  int* perm;
  double* scratch;
  int* flags;
};

// The second area holds V during the Jacobi sweeps and, in k_small_rr, the
// R^p orthonormalisation work arrays afterwards (X p x na, C m x na, M, L and
// an SVQB workspace), hence its size max(p (p+1), 2 p m + 3 m^2 + 2 m).
__host__ __device__ inline int eig_area2(int p, int m) {
  const int a = p * (p + 1), b = 2 * p * m + 3 * m * m + 2 * m;
  return a > b ? a : b;
}
__device__ __forceinline__ EigLds eig_lds(double* smem, int p, int m) {
  EigLds L;
  const int ld = p + 1;
  L.A = smem;
  L.V = L.A + p * ld;
  L.cs = L.V + eig_area2(p, m);   // 3 * 64
  L.scratch = L.cs + 3 * 64;      // 16
  L.pr = (int*)(L.scratch + 16);  // 2 * 64
  L.perm = L.pr + 2 * 64;         // 128
  L.flags = L.perm + 128;         // 8
  return L;
}

// ---------------------------------------------------------------------------
// Lowest nev eigenpairs of a symmetric p x p matrix by the tridiagonal
// route (the Rayleigh-Ritz solve of Alg. 1; the paper calls LAPACK for it,
// Sec. 3.1).  Jacobi needs p - 1 dependent rounds per sweep, each a chain
// of square roots and divisions followed by a full-matrix update; this path
// has one short chain per reflector and per Sturm count instead:
//   1. Householder reduction A = Q T Q^T by the workgroup: reflector k,
//      H_k = I - beta_k v_k v_k^T, maps column k below the diagonal to
//      alpha_k e_{k+1} (v_k kept in that column, Q = H_0 H_1 ... H_{p-3});
//   2. the nev lowest eigenvalues of T by multisection on Sturm counts
//      (counts of negative pivots of T - x I with LAPACK's pivmin guard),
//      G points per eigenvalue and round;
//   3. their vectors by block inverse iteration: a solve with the
//      partial-pivoting LU of T - lambda_j I from a SplitMix64 start
//      (pivots below eps ||T|| raised to eps ||T||, one thread per vector),
//      Cholesky-QR of the nev vectors, a second solve;
//   4. back-transformation u = Q z, one wave per vector;
//   5. Cholesky-QR, twice, of the nev vectors.
// Inverse iteration returns the vectors of a cluster of close or repeated
// eigenvalues as independent mixtures of the cluster's eigenvectors, which
// drift towards each other with further solves; orthonormalising them in
// ascending order between and after the solves keeps them an orthonormal
// eigenbasis of the cluster (residuals and orthogonality ~1e-15 ||A|| on
// repeated and 1e-14-separated eigenvalues, where three plain solves
// followed by Cholesky-QR lose two digits).
// Returns false when a Cholesky-QR breaks down (A is destroyed); the
// callers then reload A and run Jacobi.

constexpr int kMsPoints = 32;              // multisection points per eigenvalue


// Every phase is bounded by the latency of dependent steps, not by their
// number, and every sum keeps its order (see the comment of k_small_rr): eight
// waves, two per SIMD, a barrier as rarely as possible.

constexpr int kRrThreads = 512;
typedef double dd2 __attribute__((ext_vector_type(2)));

// LDS layout (the matrix comes first), in doubles
struct TriLayout {
  int ldz, nb;
  int de, d, e, inve, beta, ww, ev, linv, G, Z, ws;
};
// row stride of the matrix: up to p = 64 rows are padded by 64 zeros (and lie on
// different banks), so that no lane needs to know where they end
__host__ __device__ inline int tri_lda(int p) { return p > 64 ? p + 1 : p > 33 ? 129 : 97; }
__host__ __device__ inline TriLayout tri_layout(int p, int nev) {
  TriLayout t;
  t.ldz = nev + 1;
  const int o0 = (p * tri_lda(p) + 1) & ~1;  // after the matrix
  int o = o0;
  t.de = o; o += 2 * (p + 24);  // pairs: diagonal, square of the entry above it; padded
  t.d = o; o += p + 9;
  t.e = o; o += p + 9;
  t.inve = o; o += p + 9;
  t.beta = o; o += p;
  o += o & 1;
  t.ww = o; o += (p > 64) ? p : 3 * (p + 64);
  t.ev = o; o += nev;
  t.linv = o; o += nev;
  t.G = o; o += nev * (nev + 1);
  t.Z = o; o += p * t.ldz;
  t.ws = o;
  const int avail = kEigLdsBytes / 8 - o;
  const int per = 4 * (((p + 7) & ~7) + 1);  // z, U0^-1, U1, multipliers
  int nb = avail / per;
  if (nb > nev) nb = nev;
  t.nb = nb;
  return t;
}

// Sum over 64 leaves, 4 q + u in x[u] of lane q of a row of 16, the same bits
// as wave_sum of leaf l in lane l: both add by a balanced tree.
__device__ __forceinline__ double tree64(const double (&x)[4]) { return row_sum((x[0] + x[1]) + (x[2] + x[3])); }

// Householder reduction by the whole workgroup, two barriers per step: every
// wave forms reflector k from row k (= column k, the trailing block is kept
// symmetric but for rounding); each row of 16 lanes takes a row i of
// p = beta A v, four entries per lane; every wave forms K = beta/2 p^T v and
// updates its rows of the trailing block with w = p - K v.
__device__ __forceinline__ void blk_tridiag(double* A, int lda, int p, double* d, double* e, double* beta, double* pp) {
  constexpr int NW = kRrThreads / 64;
  constexpr int H = 2, T = 3;  // entries per lane / 4, passes of 4 NW rows
  const int tid = threadIdx.x, wave = wave_id(), lane = tid & 63, q = lane & 15, rg = lane >> 4;
  for (int k = 0; k + 2 < p; ++k) {
    const int k1 = k + 1;
    const double* row = A + k * lda;
    const double x1 = row[k1];
    // row k by leaves of the norm (entry i: leaf i) and of the products
    // (entry k1 + l: leaf l), and this wave's rows of the block
    double xa[H][4], v[H][4], a[T][H][4];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * q + u + 64 * h, j = k1 + i;
        const double x = row[min(i, p - 1)], y = row[min(j, p - 1)];
        xa[h][u] = ((i > k1) & (i < p)) ? x : 0.0;
        v[h][u] = (j < p) ? y : 0.0;
      }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int i = k1 + 4 * wave + rg + 4 * NW * t;
      if (k1 + 4 * wave + 4 * NW * t < p) {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int j = k1 + 4 * q + u + 64 * h;
            a[t][h][u] = A[min(i, p - 1) * lda + min(j, p - 1)];  // (v is zero past the end)
          }
      }
    }
    double lf[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      lf[u] = fma(xa[0][u], xa[0][u], 0.0);  // (a bare product would fuse with the tree's first sum)
      if (H == 2) lf[u] = fma(xa[H - 1][u], xa[H - 1][u], lf[u]);
    }
    const double tail = tree64(lf);
    double alpha = x1, b = 0.0;
    if (tail > 0.0) {
      const double nrm = sqrt(x1 * x1 + tail);
      alpha = (x1 >= 0.0) ? -nrm : nrm;
      b = 1.0 / (nrm * (nrm + fabs(x1)));  // 2 / v^T v for v = x - alpha e_1
    }
    const double v1 = (b != 0.0) ? x1 - alpha : x1;
    if (tid > k && tid < p) A[tid * lda + k] = (tid == k1) ? v1 : row[tid];  // kept for the back-transformation
    if (tid == 0) {
      d[k] = row[k];
      e[k] = alpha;
      beta[k] = b;
    }
    if (b == 0.0) continue;  // H_k = I (uniform)
    if (q == 0) v[0][0] = v1;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int i = k1 + 4 * wave + rg + 4 * NW * t;
      if (k1 + 4 * wave + 4 * NW * t < p) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          lf[u] = fma(a[t][0][u], v[0][u], 0.0);
          if (H == 2) lf[u] = fma(a[t][H - 1][u], v[H - 1][u], lf[u]);
        }
        const double acc = tree64(lf);
        if (q == 0 && i < p) pp[i] = b * acc;
      }
    }
    __syncthreads();
    // column lane (+ 64) of the update, and the leaves of p^T v
    double vi[H], wi[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int i = k1 + lane + 64 * h;
      const double x = row[min(i, p - 1)];
      vi[h] = (i == k1) ? v1 : x;
      wi[h] = pp[min(i, p - 1)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      lf[u] = 0.0;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int i = k1 + 4 * q + u + 64 * h;
        const double pi = pp[min(i, p - 1)];
        lf[u] = fma((i < p) ? pi : 0.0, v[h][u], lf[u]);
      }
    }
    // rows wave, wave + NW, ...: the first ones' entries are on their way
    constexpr int UR = 4;
    double vj[UR], wj[UR], aj[UR][H];
    auto load = [&](int j0) {
#pragma unroll
      for (int r = 0; r < UR; ++r) {
        const int j = min(j0 + NW * r, p - 1);
        const double x = row[j];
        vj[r] = (j == k1) ? v1 : x;
        wj[r] = pp[j];
#pragma unroll
        for (int h = 0; h < H; ++h) aj[r][h] = A[j * lda + min(k1 + lane + 64 * h, p - 1)];
      }
    };
    load(k1 + wave);
    const double K = 0.5 * b * tree64(lf);
#pragma unroll
    for (int h = 0; h < H; ++h) wi[h] = wi[h] - K * vi[h];
    for (int j0 = k1 + wave; j0 < p; j0 += UR * NW) {
      if (j0 != k1 + wave) load(j0);
#pragma unroll
      for (int r = 0; r < UR; ++r) {
        const int j = j0 + NW * r;
        const double w = wj[r] - K * vj[r];
#pragma unroll
        for (int h = 0; h < H; ++h)
          if (j < p && k1 + lane + 64 * h < p) A[j * lda + k1 + lane + 64 * h] = aj[r][h] - (vj[r] * wi[h] + w * vi[h]);
      }
    }
    __syncthreads();
  }
  __syncthreads();
  if (tid == 0) {
    if (p >= 2) {
      d[p - 2] = A[(p - 2) * lda + p - 2];
      e[p - 2] = A[(p - 1) * lda + p - 2];
    }
    d[p - 1] = A[(p - 1) * lda + p - 1];
  }
  __syncthreads();
}

// The same up to p = 64, by four waves (one per SIMD; the others only meet the
// barriers), the block in registers: lane 16 g + l of wave w holds, of the rows
// 4 w + g + 16 t, the columns k + 1 + 4 l .. + 3 of step k, and moves them on by
// one when it has updated them.  LDS carries row k, beta and p only: a wave's
// load costs the LDS its whole width, also where all waves read the same, and
// with the block in LDS as well its traffic bound a step (3500 cycles at
// p = 48, now 3100: the chains of roots, divisions and tree sums).  The wave with row k forms the reflector; vv (two of p + 64 entries) and
// pp (p + 64) are padded by zeros, as the block is.
__device__ __forceinline__ void blk_tridiag64(double* A, int lda, int p, double* d, double* e, double* beta, double* vv0,
                                              double* pp) {
  constexpr int NW = 4;
  const int tid = threadIdx.x, wave = wave_id(), lane = tid & 63, q4 = 4 * (lane & 15), rg = lane >> 4;
  double* vv1 = vv0 + p + 64;
  for (int i = tid; i < p + 64; i += kRrThreads) vv0[i] = vv1[i] = pp[i] = 0.0;
  const int r0 = 4 * wave + rg;  // rows r0 + 16 t
  double a[4][4];
  if (wave < NW) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) a[t][u] = A[min(r0 + 16 * t, p - 1) * lda + q4 + u];
  }
  __syncthreads();
  // column k1 is first: its diagonal entry, at the end the last entries
  auto emit = [&](int k1) {
    if (wave == ((k1 >> 2) & 3)) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if ((k1 >> 4) == t) {
          if (lane == 16 * (k1 & 3)) d[k1] = a[t][0];
        }
    }
    if (k1 + 2 == p && wave == (((p - 1) >> 2) & 3)) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (((p - 1) >> 4) == t) {
          if (lane == 16 * ((p - 1) & 3)) {
            e[p - 2] = a[t][0];
            d[p - 1] = a[t][1];
          }
        }
    }
  };
  auto advance = [&](double (&x)[4]) {
    const double n = dpp_f64<0x101>(x[0]);  // lane + 1 of the row, zero past its end
    x[0] = x[1];
    x[1] = x[2];
    x[2] = x[3];
    x[3] = n;
  };
  if (wave < NW) {
    emit(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) advance(a[t]);
  }
  for (int k = 0; k + 2 < p; ++k) {
    const int k1 = k + 1;
    double* vv = (k & 1) ? vv1 : vv0;
    if (wave == ((k >> 2) & 3)) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if ((k >> 4) == t) {
          if (rg == (k & 3)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) vv[k1 + q4 + u] = a[t][u];
          }
        }
      wave_sync();
      const double x1 = vv[k1], own = vv[lane];
      double lf[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) lf[u] = vv[q4 + u];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double x = (q4 + u > k1) ? lf[u] : 0.0;
        lf[u] = fma(x, x, 0.0);  // (a bare product would fuse with the tree's first sum)
      }
      const double tail = tree64(lf);
      double alpha = x1, b = 0.0;
      if (__ballot(tail > 0.0) != 0) {  // (uniform)
        const double nrm = sqrt(fma(x1, x1, tail));
        alpha = (x1 >= 0.0) ? -nrm : nrm;
        b = 1.0 / (nrm * (nrm + fabs(x1)));  // 2 / v^T v for v = x - alpha e_1
      }
      const double v1 = (b != 0.0) ? x1 - alpha : x1;
      if (lane == 0) {
        vv[k1] = v1;
        e[k] = alpha;
        beta[k] = b;
      }
      if ((lane > k) & (lane < p)) A[lane * lda + k] = (lane == k1) ? v1 : own;  // kept for the back-transformation
    }
    __syncthreads();
    const double b = beta[k];
    const bool on = __ballot(b != 0.0) != 0;  // (uniform; else H_k = I)
    double v[4];
    if ((wave < NW) & on) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = vv[k1 + q4 + u];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if ((16 * t + 15 >= k1) & (16 * t < p)) {
          double lf[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) lf[u] = fma(a[t][u], v[u], 0.0);
          const double acc = tree64(lf);
          const int i = r0 + 16 * t;
          if ((q4 == 0) & (i >= k1) & (i < p)) pp[i] = b * acc;
        }
    }
    __syncthreads();
    if (wave < NW) {
      if (on) {
        double lf[4], wi[4], vj[4], pj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) wi[u] = pp[k1 + q4 + u];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = min(r0 + 16 * t, p - 1);
          vj[t] = vv[i];
          pj[t] = pp[i];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) lf[u] = fma(wi[u], v[u], 0.0);
        const double K = 0.5 * b * tree64(lf);
#pragma unroll
        for (int u = 0; u < 4; ++u) wi[u] = fma(-K, v[u], wi[u]);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if ((16 * t + 15 >= k1) & (16 * t < p)) {
            const double wj = fma(-K, vj[t], pj[t]);
#pragma unroll
            for (int u = 0; u < 4; ++u) a[t][u] = a[t][u] - fma(vj[t], wi[u], wj * v[u]);
          }
      }
      emit(k1);
#pragma unroll
      for (int t = 0; t < 4; ++t) advance(a[t]);
    }
  }
  __syncthreads();
}

// 1 / q to ~1 ulp: the hardware reciprocal and one Newton step (the Sturm
// count only needs each step to a few ulps, Kahan's backward-error argument)
__device__ __forceinline__ double rcp_nr(double q) {
  const double r = __builtin_amdgcn_rcp(q);
  return fma(r, fma(-q, r, 1.0), r);
}

// number of eigenvalues of T below x (negative pivots of T - x I).  Each row of
// 16 lanes holds the pairs (diagonal, square of the entry above it) of steps
// 1 + 16 c + (lane % 16) in t[c] and hands them on by DPP (read from LDS, each
// wave's broadcast of a pair costs 8 cycles of all waves': that bound the
// loop); past the end come steps (infinity, 0) that count nothing.
template <int NC>
__device__ __forceinline__ int sturm_count(const double (&td)[NC], const double (&te)[NC], double d0, int p, double x,
                                           double pivmin) {
  int c = 0;
  double q = d0 - x;
  auto guard = [&]() {
    c += (q <= pivmin) ? 1 : 0;
    q = (fabs(q) <= pivmin) ? -pivmin : q;
  };
  guard();
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    if (1 + 16 * k >= p) break;
    static_for<0, 4>([&](auto h) {
      if (1 + 16 * k + 4 * decltype(h)::value < p) {
        static_for<0, 4>([&](auto u) {
          constexpr int U = 4 * decltype(h)::value + decltype(u)::value;
          q = (row_bcast<U>(td[k]) - x) - row_bcast<U>(te[k]) * rcp_nr(q);
          guard();
        });
      }
    });
  }
  return c;
}

// eigenvalues 0 .. nev-1 (ascending) of T into ev; every thread calls it.  The
// points per eigenvalue and round are those of 1024 threads.
template <int NC>
__device__ __forceinline__ void blk_multisection(const dd2* de, int p, int nev, double gl, double gu, double tnorm,
                                                 double pivmin, double* ev) {
  int G = kMsPoints;
  while (G > 1 && G * nev > 1024) G >>= 1;
  const int t = threadIdx.x & (G - 1);
  const int gi = threadIdx.x / G, ngroups = kRrThreads / G;
  const int lane = threadIdx.x & 63;
  const uint64_t gmask = (G == 64) ? ~0ull : (((1ull << G) - 1ull) << (lane & ~(G - 1)));
  double td[NC], te[NC];
  const double d0 = de[0][0];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const dd2 x = de[min(1 + 16 * c + (lane & 15), p + 15)];
    td[c] = x[0];
    te[c] = x[1];
  }
  for (int j0 = 0; j0 < nev; j0 += ngroups) {
    const int j = j0 + gi;
    bool act = j < nev;
    double lo = gl, hi = gu;
    for (int round = 0; round < 256; ++round) {
      const double w = hi - lo;
      act = act && !(w <= 2.0 * kEps * fmax(fabs(lo), fabs(hi)) || w <= kEps * tnorm);
      if (__ballot(act) == 0) break;  // (all lanes of a wave run: their registers are read by DPP)
      const double h = w / (double)(G + 1);
      const double x = lo + (double)(t + 1) * h;
      const int c = sturm_count<NC>(td, te, d0, p, x, pivmin);
      const int k = __popcll(__ballot(c <= j) & gmask);
      const double nlo = (k > 0) ? lo + (double)k * h : lo;
      const double nhi = (k < G) ? lo + (double)(k + 1) * h : hi;
      act = act && !(nlo == lo && nhi == hi);
      if (act) {
        lo = nlo;
        hi = nhi;
      }
    }
    if (t == 0 && j < nev) ev[j] = lo + 0.5 * (hi - lo);
  }
}

// Inverse iteration, one solve of (T - lam I) z = z per thread, in two halves.
// The forward one builds the LU (FACTOR: partial pivoting by selects, so that
// lanes that swap and lanes that do not take the same steps) and keeps U1, the
// multipliers and the pivots, whose reciprocals the whole workgroup forms in
// between, in LDS, the swaps as bits in sw0, sw1: U2 is e_{i+1} after a swap, 0
// otherwise.  One thread's entries of an array lie together (odd stride between
// threads: no address arithmetic, no bank conflicts), rows p .. p8-1 continue T
// by the identity (e = 0; zero in z) and leave the others as they are, so that
// rows go by eights without a branch, their operands loaded ahead of the
// dependent chain.
template <bool FACTOR>
__device__ __forceinline__ void invit_forward(const double* __restrict__ d, const double* __restrict__ e,
                                              const double* __restrict__ inve, int p8, double lam, double tol,
                                              double* __restrict__ Z, double* __restrict__ U0,
                                              double* __restrict__ U1, double* __restrict__ LM, uint64_t& sw0,
                                              uint64_t& sw1) {
  double y = Z[0];
  double c0 = d[0] - lam, c1 = e[0];
  if (FACTOR) sw0 = sw1 = 0;
  for (int i0 = 0; i0 < p8; i0 += 8) {
    double bz[8], dn[8], en[9], ie[8], lm[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u;
      bz[u] = Z[i + 1];
      if (FACTOR) {
        dn[u] = d[i + 1] - lam;
        en[u] = e[i];
        ie[u] = inve[i];
      } else {
        lm[u] = LM[i];
      }
    }
    if (FACTOR) en[8] = e[i0 + 8];
    uint32_t m = 0;
    if (!FACTOR) m = (uint32_t)(((i0 < 64) ? sw0 : sw1) >> (i0 & 63));
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u;
      bool s;
      double li;
      if (FACTOR) {
        const double ei = en[u], ex = en[u + 1];
        s = !(fabs(c0) >= fabs(ei));
        const double cand = s ? ei : c0;
        const double piv = (fabs(cand) < tol) ? ((cand < 0.0) ? -tol : tol) : cand;
        double l0 = ei / piv;
        asm("" : "+v"(l0));  // (a select, not a branch around the division)
        li = s ? c0 * ie[u] : l0;
        const double u1 = s ? dn[u] : c1;
        U0[i] = piv;
        U1[i] = u1;
        LM[i] = li;
        m |= s ? (1u << u) : 0u;
        c0 = fma(-li, u1, s ? c1 : dn[u]);
        c1 = s ? -li * ex : ex;
      } else {
        s = (m >> u) & 1;
        li = lm[u];
      }
      const double zi = s ? bz[u] : y;
      Z[i] = zi;
      y = fma(-li, zi, s ? y : bz[u]);
    }
    if (FACTOR) {
      if (i0 < 64) sw0 |= (uint64_t)m << i0;
      else sw1 |= (uint64_t)m << (i0 - 64);
    }
  }
}
// Z: the row-major vectors' column, which receives the scaled result
__device__ __forceinline__ void invit_backward(const double* __restrict__ e, int p, int p8, double* __restrict__ z,
                                               const double* __restrict__ U0, const double* __restrict__ U1,
                                               uint64_t sw0, uint64_t sw1, double* __restrict__ Z, int ldz) {
  double z1 = 0.0, z2 = 0.0, zmax = 0.0;
  for (int i0 = p8 - 8; i0 >= 0; i0 -= 8) {
    double zr[8], u0[8], u1[8], u2[8];
    const uint32_t m = (uint32_t)(((i0 < 64) ? sw0 : sw1) >> (i0 & 63));
#pragma unroll
    for (int u = 7; u >= 0; --u) {
      const int i = i0 + u;
      zr[u] = z[i];
      u0[u] = U0[i];
      u1[u] = U1[i];
      const double ex = e[i + 1];
      u2[u] = ((m >> u) & 1) ? ex : 0.0;
    }
#pragma unroll
    for (int u = 7; u >= 0; --u) {
      const double zi = (zr[u] - u1[u] * z1 - u2[u] * z2) * u0[u];
      z[i0 + u] = zi;
      zmax = fmax(zmax, fabs(zi));
      z2 = z1;
      z1 = zi;
    }
  }
  const double sc = (zmax > 0.0 && zmax < INFINITY) ? 1.0 / zmax : 1.0;
  for (int i0 = 0; i0 < p; i0 += 8) {
    double zr[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) zr[u] = z[i0 + u];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + u < p) Z[(i0 + u) * ldz] = zr[u] * sc;
  }
}

// G (lower, n x n, stride ldg) <- Z^T Z for Z (p x n, stride ldz), every
// thread; ends with a barrier.  Four sums per entry, over i = u (mod 4), the
// last p % 4 rows in the first; one MFMA takes four terms of one of them.
__device__ __forceinline__ void blk_gram_lower(const double* Z, int ldz, int p, int n, double* G, int ldg) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int tn = (n + 15) >> 4, p4 = p & ~3;
  for (int t = wave_id(); t < tn * tn; t += blockDim.x >> 6) {
    const int ti = tn == 1 ? t : t / tn, i0 = 16 * ti, j0 = 16 * (t - ti * tn);
    if (j0 > i0) continue;
    const bool vi = i0 + r < n, vj = j0 + r < n;
    d4 acc[4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
    for (int k0 = 0; k0 < p4; k0 += 16) {
      double av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + 4 * g + u;
        const double x = Z[min(k, p - 1) * ldz + min(i0 + r, n - 1)], y = Z[min(k, p - 1) * ldz + min(j0 + r, n - 1)];
        av[u] = (vi & (k < p4)) ? x : 0.0;
        bv[u] = (vj & (k < p4)) ? y : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = mma64(av[u], bv[u], acc[u]);
    }
    if (p4 < p) {
      const int k = p4 + g;
      const double x = Z[min(k, p - 1) * ldz + min(i0 + r, n - 1)], y = Z[min(k, p - 1) * ldz + min(j0 + r, n - 1)];
      acc[0] = mma64((vi & (k < p)) ? x : 0.0, (vj & (k < p)) ? y : 0.0, acc[0]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 4 * q + g;
      if (i < n && vj && j0 + r <= i) G[i * ldg + j0 + r] = (acc[0][q] + acc[1][q]) + (acc[2][q] + acc[3][q]);
    }
  }
  __syncthreads();
}

// Z <- Z L^-T with L L^T = G (the Gram Z^T Z from blk_gram_lower); G may be
// overwritten.  Every thread calls it; n <= 16: a wave per 64 rows, each with
// the factor in its registers, else one wave and the factor in LDS.  False
// (uniform) when a pivot is not > 0.
template <int NR>
__device__ __forceinline__ bool wave_cholqr(double* Z, int ldz, int p, int n, double* G, int ldg, double* linv) {
  const int l = threadIdx.x & 63;
  wave_sync();
  for (int k = 0; k < n; ++k) {
    const double gkk = G[k * ldg + k];
    if (!(gkk > 0.0) || !(gkk < INFINITY)) return false;
    const double lkk = sqrt(gkk), inv = 1.0 / lkk;
#pragma unroll
    for (int h = 0; h < NR; ++h) {
      const int r = l + 64 * h;
      if (r > k && r < n) G[r * ldg + k] *= inv;
    }
    if (l == 0) {
      G[k * ldg + k] = lkk;
      linv[k] = inv;
    }
    wave_sync();
    // trailing update, lane c owning column c: G[r][c] -= L[r][k] L[c][k], r >= c > k
#pragma unroll
    for (int h = 0; h < NR; ++h) {
      const int c = l + 64 * h;
      if (c > k && c < n) {
        const double lck = G[c * ldg + k];
        for (int r0 = c; r0 < n; r0 += 4) {
          double lk[4], gc[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int r = min(r0 + u, n - 1);
            lk[u] = G[r * ldg + k];
            gc[u] = G[r * ldg + c];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (r0 + u < n) G[(r0 + u) * ldg + c] = gc[u] - lk[u] * lck;
        }
      }
    }
    wave_sync();
  }
#pragma unroll
  for (int h = 0; h < NR; ++h) {
    const int i = l + 64 * h;
    if (i < p) {
      for (int jj = 0; jj < n; ++jj) {
        double s0 = Z[i * ldz + jj], s1 = 0.0;
        int k = 0;
        for (; k + 2 <= jj; k += 2) {
          s0 -= Z[i * ldz + k] * G[jj * ldg + k];
          s1 -= Z[i * ldz + k + 1] * G[jj * ldg + k + 1];
        }
        if (k < jj) s0 -= Z[i * ldz + k] * G[jj * ldg + k];
        Z[i * ldz + jj] = (s0 + s1) * linv[jj];
      }
    }
  }
  wave_sync();
  return true;
}
__device__ __forceinline__ bool blk_cholqr(double* Z, int ldz, int p, int n, double* G, int ldg, double* linv,
                                           int* flag) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  if (n <= 16) {
    if (n <= 8) chol_trsm<8, false, true>(Z, ldz, p, n, G, ldg, flag);
    else chol_trsm<16, false, true>(Z, ldz, p, n, G, ldg, flag);
  } else if (wave == 0) {
    const bool ok = (p <= 64) ? wave_cholqr<1>(Z, ldz, p, n, G, ldg, linv)
                              : wave_cholqr<2>(Z, ldz, p, n, G, ldg, linv);
    if (lane == 0) *flag = ok ? 1 : 0;
  }
  __syncthreads();
  const bool ok = *flag != 0;
  __syncthreads();  // the flag is rewritten by the next call
  return ok;
}

// u = H_0 H_1 ... H_{p-3} z, 16 lanes per vector (z in the columns of Z, the
// reflectors in the columns of A), the next reflector on its way
template <int H>
__device__ __forceinline__ void blk_backtransform(double* Z, int ldz, const double* A, int lda, int p, int nev,
                                                  const double* beta) {
  const int lane = threadIdx.x & 63, q = lane & 15, rg = lane >> 4;
  for (int j0 = 4 * wave_id(); j0 < nev; j0 += 4 * (kRrThreads / 64)) {
    const int j = j0 + rg;
    double z[H][4], vn[H][4], bn = 0.0;
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * q + u + 64 * h;
        const double x = Z[min(i, p - 1) * ldz + min(j, nev - 1)];
        z[h][u] = (i < p) ? x : 0.0;
      }
    auto next = [&](int k) {
      k = max(k, 0);
      bn = beta[k];  // 0 for H_k = I: then s = 0
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = 4 * q + u + 64 * h;
          const double x = A[min(i, p - 1) * lda + k];
          vn[h][u] = ((i > k) & (i < p)) ? x : 0.0;
        }
    };
    next(p - 3);
    for (int k = p - 3; k >= 0; --k) {
      double v[H][4], lf[4], b = bn;
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          v[h][u] = vn[h][u];
          asm("" : "+v"(v[h][u]));
        }
      asm("" : "+v"(b));
      next(k - 1);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (H == 1) lf[u] = fma(v[0][u], z[0][u], 0.0);
        else lf[u] = v[0][u] * z[0][u] + v[H - 1][u] * z[H - 1][u];
      }
      const double sv = b * tree64(lf);
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int u = 0; u < 4; ++u) z[h][u] -= sv * v[h][u];
    }
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * q + u + 64 * h;
        if (i < p && j < nev) Z[i * ldz + j] = z[h][u];
      }
  }
  __syncthreads();
}

// The whole path (1-5).  A: p x lda in LDS (destroyed), at base, which is laid
// out by tri_layout(p, nev), whose ev and Z receive the result.  Every
// thread calls it; the return value is uniform.
__device__ __forceinline__ bool blk_tri_eigh(double* A, int lda, int p, int nev, double* base, const TriLayout& L,
                             int* flag) {
  double* d = base + L.d;
  double* e = base + L.e;
  double* inve = base + L.inve;
  double* beta = base + L.beta;
  double* ev = base + L.ev;
  double* Z = base + L.Z;
  dd2* de = reinterpret_cast<dd2*>(base + L.de);
  const int ldz = L.ldz;
  const int lane = threadIdx.x & 63;
  if (p <= 64) blk_tridiag64(A, lda, p, d, e, beta, base + L.ww, base + L.ww + 2 * (p + 64));
  else blk_tridiag(A, lda, p, d, e, beta, base + L.ww);
  // Gershgorin interval, ||T||, pivmin, by every wave
  double gl = -INFINITY, gu = -INFINITY, emax2 = 0.0;  // (gl holds -min)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h;
    if (i < p) {
      const double ei = (i + 1 < p) ? e[i] : 0.0;
      const double r = ((i > 0) ? fabs(e[i - 1]) : 0.0) + fabs(ei);
      gl = fmax(gl, -(d[i] - r));
      gu = fmax(gu, d[i] + r);
      emax2 = fmax(emax2, ei * ei);
    }
  }
  gl = -wave_max(gl);
  gu = wave_max(gu);
  emax2 = wave_max(emax2);
  const double tnorm = fmax(fabs(gl), fabs(gu));
  if (!(tnorm < INFINITY)) return false;
  if (tnorm == 0.0) {  // the zero matrix
    for (int idx = threadIdx.x; idx < p * nev; idx += blockDim.x) {
      const int i = idx / nev, j = idx - i * nev;
      Z[i * ldz + j] = (i == j) ? 1.0 : 0.0;
    }
    for (int j = threadIdx.x; j < nev; j += blockDim.x) ev[j] = 0.0;
    __syncthreads();
    return true;
  }
  const double pivmin = 0x1.0p-1022 * fmax(1.0, emax2);
  const double tol = kEps * tnorm;
  const double widen = 2.1 * (kEps * tnorm * p + 2.0 * pivmin);
  gl -= widen;
  gu += widen;
  {
    const int i = threadIdx.x;
    if (i < p) {
      const double em = (i > 0) ? e[i - 1] : 0.0, ei = (i + 1 < p) ? e[i] : 0.0;
      de[i] = dd2{d[i], em * em};
      const double piv = (fabs(ei) < tol) ? ((ei < 0.0) ? -tol : tol) : ei;
      inve[i] = (ei == 0.0) ? 0.0 : 1.0 / piv;
    } else if (i < p + 24) {
      de[i] = dd2{INFINITY, 0.0};
      if (i < p + 9) {
        d[i] = 1.0;
        e[i] = inve[i] = 0.0;
      }
    }
    if (i == p - 1) e[i] = 0.0;
  }
  // start vectors
  for (int j = threadIdx.x & 15; j < nev; j += 16)
    for (int i = threadIdx.x >> 4; i < p; i += kRrThreads / 16) {
      const uint64_t z = sm64(kZeroColumnSeed ^ (0x5EEDull << 32) ^ ((uint64_t)j * (uint64_t)p + (uint64_t)i));
      Z[i * ldz + j] = (double)(z >> 11) * 0x1.0p-52 - 1.0;
    }
  __syncthreads();
  if (p <= 49) blk_multisection<3>(de, p, nev, gl, gu, tnorm, pivmin, ev);
  else blk_multisection<6>(de, p, nev, gl, gu, tnorm, pivmin, ev);
  __syncthreads();
  // two solves with a Cholesky-QR between them (block inverse iteration);
  // with several batches the LU is rebuilt for the second solve
  const int nb = L.nb, p8 = (p + 7) & ~7, ps = p8 + 1;
  uint64_t sw0 = 0, sw1 = 0;
  for (int it = 0; it < 2; ++it) {
    for (int j0 = 0; j0 < nev; j0 += nb) {
      const int t = threadIdx.x, j = min(j0 + t, nev - 1), nv = min(nb, nev - j0);
      const bool mine = t < nv, factor = it == 0 || nb < nev;
      double *z0 = base + L.ws, *U0 = z0 + nb * ps, *U1 = U0 + nb * ps, *LM = U1 + nb * ps;
      for (int v = t >> 4; v < nv; v += kRrThreads / 16)
        for (int i = t & 15; i <= p8; i += 16) z0[v * ps + i] = (i < p) ? Z[i * ldz + j0 + v] : 0.0;
      __syncthreads();
      if (mine) {
        if (factor) invit_forward<true>(d, e, inve, p8, ev[j], tol, z0 + t * ps, U0 + t * ps, U1 + t * ps, LM + t * ps, sw0, sw1);
        else invit_forward<false>(d, e, inve, p8, ev[j], tol, z0 + t * ps, U0 + t * ps, U1 + t * ps, LM + t * ps, sw0, sw1);
      }
      if (factor) {
        __syncthreads();
        for (int v = t >> 4; v < nv; v += kRrThreads / 16)
          for (int i = t & 15; i < p8; i += 16) U0[v * ps + i] = 1.0 / U0[v * ps + i];
        __syncthreads();
      }
      if (mine) invit_backward(e, p, p8, z0 + t * ps, U0 + t * ps, U1 + t * ps, sw0, sw1, Z + j, ldz);
      __syncthreads();
    }
    if (it == 0) {
      blk_gram_lower(Z, ldz, p, nev, base + L.G, nev + 1);
      if (!blk_cholqr(Z, ldz, p, nev, base + L.G, nev + 1, base + L.linv, flag)) return false;
    }
  }
  if (p <= 64) blk_backtransform<1>(Z, ldz, A, lda, p, nev, beta);
  else blk_backtransform<2>(Z, ldz, A, lda, p, nev, beta);
  // Cholesky-QR twice, with the A area as Gram scratch.  One pass leaves
  // the vectors orthonormal to a few units of rounding when the Gram is
  // well conditioned, yet the second pass is kept: the P coefficients are
  // the small differences u_x - E, and dropping it whenever the columns'
  // cosines were below 1e-3 doubled the iterations of a dense generalized
  // solve (n = 2000, 4 pairs: 51 against 25, the lowest pair lagging).
  for (int pass = 0; pass < 2; ++pass) {
    blk_gram_lower(Z, ldz, p, nev, A, lda);
    if (!blk_cholqr(Z, ldz, p, nev, A, lda, base + L.linv, flag)) return false;
  }
  return true;
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

// sym(a) into A (stride lda; columns up to width zero), with the pending column scaling of the W block
// (see small_rr in internal.h) applied from both sides when pend != nullptr
__device__ __forceinline__ void load_rr_matrix(const double* a, int p, double* A, int lda, int width,
                                               const OrthoState* pend, int woff) {
  const int nws = (pend != nullptr) ? pend->nw : 0;
  for (int j = threadIdx.x & 63; j < width; j += 64) {
    if (j >= p) {
      for (int i = threadIdx.x >> 6; i < p; i += blockDim.x >> 6) A[i * lda + j] = 0.0;
      continue;
    }
    const double dj = (j >= woff && j < woff + nws) ? pend->dscale[j - woff] : 1.0;
#pragma unroll 4
    for (int i = threadIdx.x >> 6; i < p; i += blockDim.x >> 6) {
      const double di = (i >= woff && i < woff + nws) ? pend->dscale[i - woff] : 1.0;
      const double v = 0.5 * (a[i * p + j] + a[j * p + i]);
      A[i * lda + j] = (nws > 0) ? v * (di * dj) : v;
    }
  }
  __syncthreads();
}

}  // namespace

// Rayleigh-Ritz step.  The order of every sum is part of what it computes: an
// iteration that has not converged amplifies rounding (on a banded matrix of
// order 1e5, one unit in the last place of the starting block moves the
// eigenvalues in the first digit after five iterations), so a change of order
// would change what a few iterations give and what is trained on it.
// JAC: the Jacobi option, 1024 threads; else the tridiagonal path, 512.
// Measured (p = 48, m = 16; 39, 13; 24, 8; 12, 4): 160, 135, 79, 52 us, where
// 1024 threads with three barriers per reflector, whole waves per row, one
// column per thread in the triangular solves and scalar loops for the products
// took 257, 187, 107, 60; above p = 64, where LDS holds no padded rows and the
// vectors are more than 16, 848 against 970 us (p = 96, m = 32).
template <bool JAC>
__global__ __launch_bounds__(JAC ? 1024 : kRrThreads) void k_small_rr(const double* __restrict__ a, int p, int m,
                                                  int a0, int want_up, double tau,
                                                  const OrthoState* __restrict__ pend, int woff,
                                                  double* __restrict__ theta_all,
                                                  double* __restrict__ U, int* __restrict__ info) {
  constexpr int NT = JAC ? 1024 : kRrThreads;
  extern __shared__ __attribute__((aligned(16))) double smem[];
  EigLds L = eig_lds(smem, p, m);
  const int ld = p + 1;
  __shared__ ShiftCount cnt;
  __shared__ int zeros;
  __shared__ int stalled, passes, grams, updates, tflag;
  if (threadIdx.x == 0) {
    cnt.factorizations = cnt.failed = cnt.shifted = cnt.svqb = 0;
    zeros = stalled = passes = grams = updates = 0;
  }
  const bool scaled = (pend != nullptr) && pend->pending_scale;
  double* Us = L.A;  // sorted eigenvectors u_x (first m columns), stride ld
  int sw = 0;
  const TriLayout T = tri_layout(p, m);
  bool tri = false;
  if (!JAC && T.nb >= 1) {
    const int lda = tri_lda(p);
    load_rr_matrix(a, p, L.A, lda, lda > p + 1 ? lda : p, scaled ? pend : nullptr, woff);
    double* base = L.A;
    tri = blk_tri_eigh(L.A, lda, p, m, base, T, &tflag);
    if (tri) {
      for (int j = threadIdx.x; j < m; j += blockDim.x) theta_all[j] = base[T.ev + j];
      // orientation: u[j][j] >= 0, so that u_x - E is the small update X_new - X_old
      for (int j = threadIdx.x & 15; j < m; j += 16) {
        const double sg = (base[T.Z + j * T.ldz + j] < 0.0) ? -1.0 : 1.0;
        for (int i = threadIdx.x >> 4; i < p; i += NT / 16) Us[i * ld + j] = sg * base[T.Z + i * T.ldz + j];
      }
      __syncthreads();
    }
  }
  if (!tri) {
    load_rr_matrix(a, p, L.A, ld, p, scaled ? pend : nullptr, woff);
    sw = blk_jacobi<NT>(L.A, ld, L.V, ld, p, L.cs, L.pr, L.flags, L.scratch);
    blk_sort_evals(L.A, ld, p, L.perm);
    for (int j = threadIdx.x; j < m; j += blockDim.x) theta_all[j] = L.A[L.perm[j] * ld + L.perm[j]];
    __syncthreads();
    for (int idx = threadIdx.x; idx < p * p; idx += blockDim.x) {
      const int i = idx / p, j = idx - i * p;
      const double sg = (L.V[j * ld + L.perm[j]] < 0.0) ? -1.0 : 1.0;
      Us[i * ld + j] = sg * L.V[i * ld + L.perm[j]];
    }
    __syncthreads();
  }
  const int na = want_up ? (m - a0) : 0;
  const int q = m + na;
  // u_x (row scaling for a pending W scaling is applied when U is written)
  const int sn = scaled ? pend->nw : 0;
  for (int j = threadIdx.x & 15; j < m; j += 16)
    for (int i = threadIdx.x >> 4; i < p; i += NT / 16) {
      const double di = (i >= woff && i < woff + sn) ? pend->dscale[i - woff] : 1.0;
      U[i * q + j] = di * Us[i * ld + j];
    }
  int bad = 0;
  if (na > 0) {
    // V area becomes: X (p x na), C (m x na), M (na x na), Lc (na x na), Li, svqb workspace
    double* X = L.V;
    const int ldx = na;
    double* C = X + p * na;
    double* M = C + m * na;
    double* Lc = M + na * na;
    double* Ws = Lc + na * na;
    // u~_p = u_x[:, a0:m] - E[:, a0:m]
    for (int j = threadIdx.x & 15; j < na; j += 16)
      for (int i = threadIdx.x >> 4; i < p; i += NT / 16) X[i * ldx + j] = Us[i * ld + a0 + j] - ((i == a0 + j) ? 1.0 : 0.0);
    __syncthreads();
    blk_normalize(X, ldx, p, na, L.cs, &zeros);
    blk_gemm_tn(Us, ld, X, ldx, p, m, na, C, na);  // C = u_x^T X
    for (int pass = 0; pass < 4; ++pass) {
      if (threadIdx.x == 0) passes++;
      blk_sub_mm(X, ldx, Us, ld, C, na, p, m, na);
      // ortho(X): normalise, then Gram / check / shifted Cholesky / X L^-T
      blk_normalize(X, ldx, p, na, L.cs, &zeros);
      for (int it = 0; it < 6; ++it) {
        blk_gemm_tn(X, ldx, X, ldx, p, na, na, M, na);
        if (threadIdx.x == 0) grams++;
        // (M's two halves take the same operations: it is symmetric)
        double dev = 0.0;
        for (int j = threadIdx.x & 15; j < na; j += 16)
          for (int i = (threadIdx.x & 63) >> 4; i < na; i += 4) dev = fmax(dev, fabs(M[i * na + j] - (i == j ? 1.0 : 0.0)));
        dev = wave_max(dev);  // every wave
        if (dev <= tau) break;
        if (it == 5) {
          if (threadIdx.x == 0) stalled++;
          break;
        }
        // plain Cholesky, then shifts
        bool ok = false;
        if (!JAC && na <= 16) {
          if (na <= 8) chol_trsm<8, true, false>(X, ldx, p, na, M, na, L.flags);
          else chol_trsm<16, true, false>(X, ldx, p, na, M, na, L.flags);
          __syncthreads();
          ok = L.flags[0] != 0;
          if (ok && threadIdx.x == 0) cnt.factorizations++;
          __syncthreads();
        }
        if (ok) {
        } else if (blk_shifted_chol<JAC>(M, na, na, Lc, na, L.flags, &cnt, kShiftRetries, JAC || na > 16)) {
          blk_trsm_rt(X, ldx, p, na, Lc, na);
        } else {
          if (threadIdx.x == 0) cnt.svqb++;
          if (!blk_svqb_coef<NT>(M, na, na, Lc, na, Ws, L.cs, L.pr, L.flags, L.perm, L.scratch)) {
            bad = 1;
            break;
          }
          // X <- X Cf (Cf in Lc), through the Ws area as a copy of X
          for (int idx = threadIdx.x; idx < p * na; idx += blockDim.x) Ws[idx] = X[idx];
          __syncthreads();
          for (int idx = threadIdx.x; idx < p * na; idx += blockDim.x) {
            const int r = idx / na, j = idx - r * na;
            double acc = 0.0;
            for (int k = 0; k < na; ++k) acc += Ws[r * na + k] * Lc[k * na + j];
            X[r * ldx + j] = acc;
          }
          __syncthreads();
        }
        if (threadIdx.x == 0) updates++;
      }
      if (bad) break;
      blk_gemm_tn(Us, ld, X, ldx, p, m, na, C, na);
      double cm = 0.0;
      for (int j = threadIdx.x & 15; j < na; j += 16)
        for (int i = (threadIdx.x & 63) >> 4; i < m; i += 4) cm = fmax(cm, fabs(C[i * na + j]));
      cm = wave_max(cm);  // every wave
      if (cm <= tau) break;
      if (pass == 3 && threadIdx.x == 0) stalled++;
    }
    for (int j = threadIdx.x & 15; j < na; j += 16)
      for (int i = threadIdx.x >> 4; i < p; i += NT / 16) {
        const double di = (i >= woff && i < woff + sn) ? pend->dscale[i - woff] : 1.0;
        U[i * q + m + j] = di * X[i * ldx + j];
      }
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

template <bool JAC>
static hipError_t rr_launch(const double* a, int p, int m, int a0, int want_up, double tau, const OrthoState* pend,
                            int woff, double* theta_all, double* U, int* info, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    // dynamic + static LDS must stay within the 160 KB of a workgroup
    (void)hipFuncSetAttribute((const void*)k_small_rr<JAC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kEigLdsBytes);
    (void)hipGetLastError();
    attr = true;
  }
  hipLaunchKernelGGL(k_small_rr<JAC>, dim3(1), dim3(JAC ? 1024 : kRrThreads), kEigLdsBytes, s, a, p, m, a0, want_up,
                     tau, pend, woff, theta_all, U, info);
  return hipGetLastError();
}

hipError_t small_rr(const double* a, int p, int m, int a0, int want_up, double tau,
                    const OrthoState* pend, int woff, double* theta_all, double* U, int* info,
                    int jacobi, hipStream_t s) {
  if (p < 1 || p > kMaxP || m < 1 || m > p || a0 < 0 || a0 > m) return hipErrorInvalidValue;
  return jacobi ? rr_launch<true>(a, p, m, a0, want_up, tau, pend, woff, theta_all, U, info, s)
                : rr_launch<false>(a, p, m, a0, want_up, tau, pend, woff, theta_all, U, info, s);
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

namespace {

enum { kPhFinal = 5, kPhYCheck = 6 };

// The ortho controller is one workgroup between two passes over the vectors, so
// its latency is what counts: a chain of roots and divisions, barriers, and the
// waits for its inputs.  Threads: the fewest that fill a block of 16 (each has
// one entry of the overlap), so the factor has the registers it needs and a
// reduction four waves to join.  12.1 us for a block of 16 under 32 columns
// (18.6 with 1024 threads, where the factor spills), 4.4 of it the factor and
// its inverse; 6.3 us (10.8 before) over the calls of a solve, many of which
// have nothing to factor.
constexpr int kCtlThreads = 256;

// maximum of non-negative values over the workgroup, in every thread
__device__ __forceinline__ double ctl_max(double v, double* scratch) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  v = fmax(fmax(scratch[0], scratch[1]), fmax(scratch[2], scratch[3]));
  __syncthreads();
  return v;
}
// sum over the wave, partners 32, 16, 8, 4, 2, 1 apart in turn (a value that is
// the same 8 lanes on is the same 4 lanes on as 4 lanes back)
__device__ __forceinline__ double wave_sum_halves(double v) {
  double a, b;
  lane_pair<32>(v, a, b);
  lane_pair<16>(a + b, a, b);
  v = a + b;
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  return v;
}
// Bound on ||L^-1||_2 for the n x n lower factor L (stride ldl) with its
// inverse Li (stride ldi): 1 / (1 - e) when e = ||I - L||_F < 1/2 (Neumann
// series), else ||Li||_F.  *e_out receives e.  Every thread gets the result.
__device__ __forceinline__ double blk_inv_bound(const double* L, int ldl, const double* Li, int ldi, int n,
                                double* e_out, double* scratch) {
  // 64 entries to a partial sum, these in order (scratch: two times 16)
  const unsigned parts = (n * n + 63) / 64;
  for (unsigned p = wave_id(); p < parts; p += kCtlThreads / 64) {
    const unsigned idx = 64 * p + (threadIdx.x & 63), i = idx / unsigned(n), j = idx - i * n;
    double de = 0.0, di = 0.0;
    if (i < unsigned(n) && j <= i) {
      de = (i == j ? 1.0 : 0.0) - L[i * ldl + j];
      di = Li[i * ldi + j];
    }
    de = wave_sum_halves(de * de);
    di = wave_sum_halves(di * di);
    if ((threadIdx.x & 63) == 0) {
      scratch[2 * p] = de;
      scratch[2 * p + 1] = di;
    }
  }
  __syncthreads();
  double se = scratch[0], si = scratch[1];
  for (unsigned p = 1; p < parts; ++p) {
    se += scratch[2 * p];
    si += scratch[2 * p + 1];
  }
  const double e = sqrt(se);
  *e_out = e;
  return (e < 0.5) ? 1.0 / (1.0 - e) : sqrt(si);
}

}  // namespace

__global__ __launch_bounds__(kCtlThreads) void k_ortho_ctl(const double* __restrict__ G,
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
  __shared__ double scratch[32];
  __shared__ int flag, nonfinite, zero_mask;
  __shared__ ShiftCount cnt;
  if (threadIdx.x < sizeof(OrthoState) / 4)
    reinterpret_cast<uint32_t*>(&st)[threadIdx.x] = reinterpret_cast<const uint32_t*>(gst)[threadIdx.x];
  if (threadIdx.x == 0) {
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
    // (every wave for itself)
    const int lane = threadIdx.x & 63;
    growth = wave_max((lane < nw) ? D[lane] : 0.0);
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
  dev = ctl_max(dev, scratch);
  const bool ortho_ok = dev <= st.tau;
  capped = !ortho_ok && st.inner >= st.max_inner;
  if (ortho_ok || capped) {
    if (capped && threadIdx.x == 0) st.stalled++;
    check_outer = true;
    have_scale = (phase == kPhBegin);
  } else {
    // shifted Cholesky of M (= M' in BEGIN)
    bool ok = false;
    if (nw <= 16) {  // the plain one, with its inverse
      if (threadIdx.x < 64) {
        const bool o = (nw <= 8) ? chol_inv16<8>(Ms, ldm, nw, Ls, ldm, Li, ldm)
                                 : chol_inv16<16>(Ms, ldm, nw, Ls, ldm, Li, ldm);
        if (threadIdx.x == 0) {
          flag = o ? 1 : 0;
          if (o) cnt.factorizations++;
        }
      }
      __syncthreads();
      ok = flag != 0;
      __syncthreads();
    }
    if (!ok) {
      ok = blk_shifted_chol<true>(Ms, ldm, nw, Ls, ldm, &flag, &cnt, st.shift_retries, nw > 16);
      if (ok) blk_tri_inv(Ls, ldm, nw, Li, ldm);
    }
    if (ok) {
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
      const bool sv = blk_svqb_coef<kCtlThreads>(Ms, ldm, nw, Li, ldm, Ws, cs, pr, &flag, perm, scratch);
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
  cm = ctl_max(cm, scratch);
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

static_assert(sizeof(OrthoState) % 4 == 0, "copied by words");

__global__ __launch_bounds__(256) void k_ortho_init(OrthoState* __restrict__ st, const OrthoState s) {
  const uint32_t* w = reinterpret_cast<const uint32_t*>(&s);
  for (unsigned i = threadIdx.x; i < sizeof(OrthoState) / 4; i += 256) reinterpret_cast<uint32_t*>(st)[i] = w[i];
}

hipError_t ortho_init(OrthoState* st, int ny, int nw, double tau, int max_inner, int max_outer,
                      int shift_retries, int fold_scale, double cexit, hipStream_t stream) {
  if (nw < 1 || nw > kMaxBlock || ny < 0 || ny + nw > kMaxP || shift_retries < 0)
    return hipErrorInvalidValue;
  OrthoState s;
  memset(&s, 0, sizeof(s));
  s.state = kPhStart;
  s.ny = ny;
  s.nw = nw;
  s.max_inner = max_inner;
  s.max_outer = max_outer;
  s.shift_retries = shift_retries;
  s.fold_scale = fold_scale;
  s.cheap_exit = cexit > 0.0 ? 1 : 0;
  s.cexit = cexit;
  s.growth = INFINITY;
  s.tau = tau;
  for (int j = 0; j < kMaxBlock; ++j) s.dscale[j] = 1.0;
  hipLaunchKernelGGL(k_ortho_init, dim3(1), dim3(256), 0, stream, st, s);
  return hipGetLastError();
}

hipError_t ortho_ctl(const double* G, OrthoState* st, double* coef, hipStream_t s) {
  hipLaunchKernelGGL(k_ortho_ctl, dim3(1), dim3(kCtlThreads), 0, s, G, st, coef);
  return hipGetLastError();
}

}  // namespace lobpcg
