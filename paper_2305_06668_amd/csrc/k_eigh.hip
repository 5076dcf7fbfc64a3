// Eigensolver of small symmetric fp64 matrices (p <= 96): lobpcg_small_eigh.
// One workgroup, everything resident in registers and LDS.  The solver's
// Rayleigh-Ritz step has a kernel of its own (k_small_rr), with the steps of
// the same path in another order: an iteration that has not converged
// amplifies rounding (on a banded matrix of order 1e5, one unit in the last
// place of the starting block moves the eigenvalues in the first digit after
// five iterations), so its operations keep their order, and what a few
// iterations give, and what is trained on it, stays as it was, bit for bit.
// 48 x 48 with all vectors: 550 us by k_small_rr's steps, 147 us here.
#include "small.h"

namespace lobpcg {

namespace {  // (k_small.hip has helpers of the same names, in its own order of operations)

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

// Workspace of the Jacobi sweeps besides A and V
struct JacobiLds {
  double cs[3 * 64];
  double scratch[16];
  int pr[2 * 64];
  int perm[128];
  int flags[8];
};

// sym(a) into A (stride lda)
__device__ __forceinline__ void load_sym(const double* a, int p, double* A, int lda) {
  for (int idx = threadIdx.x; idx < p * p; idx += blockDim.x) {
    const int i = idx / p, j = idx - i * p;
    A[i * lda + j] = 0.5 * (a[i * p + j] + a[j * p + i]);
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Eigenpairs of a symmetric p x p matrix by the tridiagonal
// route (as the Rayleigh-Ritz solve of Alg. 1, for which the paper calls
// LAPACK, Sec. 3.1), by one workgroup of four waves:
//   1. Householder reduction A = Q T Q^T: reflector k,
//      H_k = I - beta_k v_k v_k^T, maps column k below the diagonal to
//      alpha_k e_{k+1} (Q = H_0 H_1 ... H_{p-2}, the last one I);
//   2. the eigenvalues of T by multisection on Sturm counts,
//      G points per eigenvalue and round;
//   3. their vectors by block inverse iteration: a solve with the
//      partial-pivoting LU of T - lambda_j I from a SplitMix64 start
//      (pivots below eps ||T|| raised to eps ||T||, one thread per vector),
//      Cholesky-QR of the vectors, a second solve;
//   4. back-transformation u = Q z, 16 lanes per vector;
//   5. Cholesky-QR, twice, of the vectors.
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

constexpr int kEigThreads = 256;

typedef double dd2 __attribute__((ext_vector_type(2)));

// LDS layout of the tridiagonal path, in doubles.  The reduction's vectors and
// the LU of the inverse iteration share `lu`.  Z and the LU have rows for p
// rounded up to 8.
struct TriLayout {
  int ldz, nb;
  int Z, ev, d, e, beta, de, vref, orth, lu;
};
constexpr int kTrans = 16 * 17;  // one wave's 16 x 16 transpose
constexpr int kRedScratch = 128 + 4 * 128;
// reflectors: rows of 64 up to p = 64 (zeros in front and behind), packed above
__host__ __device__ inline int ref_doubles(int p) { return p <= 64 ? 64 * p : p * (p - 1) / 2; }
__host__ __device__ inline TriLayout tri_layout(int p) {
  TriLayout t;
  const int p8 = (p + 7) & ~7;
  t.ldz = p | 1;
  int o = 0;
  t.Z = o; o += p8 * t.ldz;
  t.ev = o; o += p;
  t.d = o; o += p8 + 1;
  t.e = o; o += p8 + 1;
  t.beta = o; o += p;
  o += o & 1;
  t.de = o; o += 2 * (p + 16);
  t.vref = o; o += ref_doubles(p);
  t.orth = o; o += 4 * kTrans + (p > 16 ? (p - 1) / 16 * 16 * 17 : 0);
  t.lu = o;
  const int avail = kEigLdsBytes / 8 - o;
  t.nb = avail / (3 * p8);  // U0^-1, U1, multipliers
  if (t.nb > p) t.nb = p;
  return t;
}
// the path runs for every p the kernel takes
static_assert(kEigLdsBytes / 8 > 96 * 97 + 4 * 98 + 2 * 112 + 96 * 95 / 2 + 4 * kTrans + 80 * 17 + kRedScratch &&
                  kEigLdsBytes / 8 > 64 * 65 + 4 * 66 + 2 * 80 + 64 * 64 + 4 * kTrans + 48 * 17 + kRedScratch,
              "LDS of the largest eigensolves");

// offset of reflector k (its entries k+1 .. p-1) in the packed store
__device__ __forceinline__ int ref_off(int p, int k) { return k * (p - 1) - k * (k - 1) / 2; }

// Householder reduction of sym(a).  Lane l of
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
__device__ __forceinline__ void reg_tridiag(const double* __restrict__ a, int p, double* d,
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
      A[h][jj] = (i < p && c < p) ? 0.5 * (a[i * p + c] + a[c * p + i]) : 0.0;
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

// Eigenvalues 0 .. p-1 (ascending) of T into ev, G lanes to each: the
// largest power of two (64 at most) with one point per thread.  More points
// per thread shorten the search by less than they add to the count loop,
// which one wave per SIMD runs at its instruction rate.  Every thread calls
// it.
__device__ __forceinline__ void blk_multisection(const dd2* de, int p, double gl, double gu, double tnorm,
                                                 double* ev) {
  int G = 64;
  while (G > 1 && G * p > kEigThreads) G >>= 1;
  const int lane = threadIdx.x & 63;
  const int t = lane & (G - 1), gi = (int)threadIdx.x / G;
  const uint64_t gmask = (G == 64) ? ~0ull : (((1ull << G) - 1ull) << (lane & ~(G - 1)));
  const double inv = 1.0 / (double)(G + 1), tp = (double)(t + 1);
  for (int j0 = 0; j0 < p; j0 += kEigThreads / G) {
    const int j = j0 + gi;
    bool act = j < p;
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
    if (t == 0 && j < p) ev[j] = lo + 0.5 * (hi - lo);
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
__device__ __forceinline__ void blk_backtransform(double* Z, int ldz, int p, const double* vref,
                                                  const double* beta) {
  const int lane = threadIdx.x & 63, s = lane & 15;
  for (int jb = 0; jb < p; jb += 16) {
    const int j = jb + 4 * wave_id() + (lane >> 4);
    double z[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int i = s + 16 * t;
      z[t] = (i < p && j < p) ? Z[i * ldz + j] : 0.0;
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
      if (i < p && j < p) Z[i * ldz + j] = z[t];
    }
  }
  __syncthreads();
}

// The whole path (1-5) on a (device, p x p); base: LDS laid out by
// tri_layout(p), whose ev and Z receive the result.  Every thread of a
// kEigThreads workgroup calls it; the return value is uniform.
__device__ __forceinline__ bool blk_tri_eigh(const double* __restrict__ a, int p, double* base,
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
  if (p <= 48) reg_tridiag<1, 12>(a, p, d, e, beta, vref, base + L.lu);
  else if (p <= 64) reg_tridiag<1, 16>(a, p, d, e, beta, vref, base + L.lu);
  else reg_tridiag<2, 24>(a, p, d, e, beta, vref, base + L.lu);
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
    for (int idx = threadIdx.x; idx < p * p; idx += kEigThreads) {
      const int i = idx / p, j = idx - i * p;
      Z[i * ldz + j] = (i == j) ? 1.0 : 0.0;
    }
    for (int j = threadIdx.x; j < p; j += kEigThreads) ev[j] = 0.0;
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
  for (int idx = threadIdx.x; idx < p8 * p; idx += kEigThreads) {
    const int i = idx / p, j = idx - i * p;
    if (i >= p) {
      Z[i * ldz + j] = 0.0;
      continue;
    }
    const uint64_t z = sm64(kZeroColumnSeed ^ (0x5EEDull << 32) ^ ((uint64_t)j * (uint64_t)p + (uint64_t)i));
    Z[i * ldz + j] = (double)(z >> 11) * 0x1.0p-52 - 1.0;
  }
  __syncthreads();
  blk_multisection(de, p, gl, gu, tnorm, ev);
  __syncthreads();
  // two solves with a Cholesky-QR between them (block inverse iteration;
  // with several batches the LU is rebuilt for the second solve), the
  // back-transformation, then Cholesky-QR twice.  One pass leaves the vectors
  // orthonormal to a few units of rounding when the Gram is well conditioned;
  // the second makes it so for the others.
  const int nb = L.nb;
  double* lu = base + L.lu;
  uint64_t sw0 = 0, sw1 = 0;
  for (int stage = 0; stage < 3; ++stage) {
    if (stage < 2) {
      for (int j0 = 0; j0 < p; j0 += nb) {
        const int t = threadIdx.x, j = j0 + t;
        if (t < nb && j < p) {
          double *u0 = lu + t, *u1 = u0 + p8 * nb, *lm = u1 + p8 * nb;
          if (stage == 0 || nb < p) tri_invit_solve<true>(d, e, p, ev[j], tol, Z, ldz, j, u0, u1, lm, nb, sw0, sw1);
          else tri_invit_solve<false>(d, e, p, ev[j], tol, Z, ldz, j, u0, u1, lm, nb, sw0, sw1);
        }
        __syncthreads();
      }
    }
    if (stage == 1) {
      if (p <= 48) blk_backtransform<3, false>(Z, ldz, p, vref, beta);
      else if (p <= 64) blk_backtransform<4, false>(Z, ldz, p, vref, beta);
      else blk_backtransform<6, true>(Z, ldz, p, vref, beta);
      for (int j = threadIdx.x; j < p; j += kEigThreads) ev[j] = __builtin_amdgcn_ldexp(ev[j], -ex);
    }
    if (!blk_cholqr(Z, ldz, p, p, base + L.orth)) return false;
  }
  return true;
}

// The same by Jacobi sweeps on all NT threads.
template <int NT>
__device__ __forceinline__ int jacobi_eigh(const double* __restrict__ a, int p, double* smem, JacobiLds& J,
                                           double* __restrict__ evals, double* __restrict__ evecs) {
  const int ld = p + 1;
  double* A = smem;
  double* V = smem + p * ld;
  load_sym(a, p, A, ld);
  const int sw = blk_jacobi<NT>(A, ld, V, ld, p, J.cs, J.pr, J.flags, J.scratch);
  blk_sort_evals(A, ld, p, J.perm);
  for (int idx = threadIdx.x; idx < p * p; idx += NT) {
    const int i = idx / p, j = idx - i * p;
    const double sg = (V[j * ld + J.perm[j]] < 0.0) ? -1.0 : 1.0;
    evecs[i * p + j] = sg * V[i * ld + J.perm[j]];
  }
  for (int j = threadIdx.x; j < p; j += NT) evals[j] = A[J.perm[j] * ld + J.perm[j]];
  return sw;
}

}  // namespace

// By rotations alone: matrices of order 1 and 2 (6 us, 15 to 19 by the
// tridiagonal path), and large ones that are diagonal up to rotations by 2^-25,
// whose squares are then below rounding: one sweep and a look.  A sweep of 16
// waves at p = 96 takes 80 us and the tridiagonal path 1160: p = 96, diagonal
// 93 us, off-diagonal parts of 1e-8 340; p = 80 76 and 267 (580).  With larger
// rotations two and three sweeps would still be the faster way, but the
// cosines' rounding adds up in the vectors (orthonormal to 2e-14, by the
// tridiagonal path to 6e-16).  What is left to that path is marked by a NaN in
// evals[0], which no result here is.
constexpr int kNearMinP = 77;
__global__ __launch_bounds__(1024) void k_small_eigh_near(const double* __restrict__ a, int p,
                                                          double* __restrict__ evals,
                                                          double* __restrict__ evecs, int* sweeps) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  __shared__ JacobiLds J;
  bool far = false;
  for (int idx = threadIdx.x; p > 2 && idx < p * p; idx += 1024) {
    const int i = idx / p, j = idx - i * p;
    if (j <= i) continue;
    const double s = 0.5 * fabs(a[i * p + j] + a[j * p + i]), di = a[i * p + i], dj = a[j * p + j];
    far |= !(s <= 0x1.0p-25 * fabs(di - dj) || s <= 0x1.0p-53 * fmin(fabs(di), fabs(dj)));
  }
  if (__syncthreads_or(far)) {
    if (threadIdx.x == 0) evals[0] = NAN;
    return;
  }
  const int sw = jacobi_eigh<1024>(a, p, smem, J, evals, evecs);
  if (threadIdx.x == 0 && sweeps != nullptr) *sweeps = sw;
}

// NEAR: after k_small_eigh_near, on what that one left
template <bool NEAR>
__global__ __launch_bounds__(kEigThreads) void k_small_eigh(const double* __restrict__ a, int p,
                                                            double* __restrict__ evals,
                                                            double* __restrict__ evecs, int* sweeps) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  __shared__ JacobiLds J;
  if (NEAR && evals[0] == evals[0]) return;
  const TriLayout T = tri_layout(p);
  if (blk_tri_eigh(a, p, smem, T)) {
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
  const int sw = jacobi_eigh<kEigThreads>(a, p, smem, J, evals, evecs);
  if (threadIdx.x == 0 && sweeps != nullptr) *sweeps = sw;
}

hipError_t small_eigh(const double* a, int p, double* evals, double* evecs, int* sweeps,
                      hipStream_t s) {
  if (p < 1 || p > kMaxP) return hipErrorInvalidValue;
  static bool attr = false;
  if (!attr) {
    for (const void* f : {(const void*)k_small_eigh<false>, (const void*)k_small_eigh<true>, (const void*)k_small_eigh_near})
      (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kEigLdsBytes);
    (void)hipGetLastError();
    attr = true;
  }
  // (a result written over the matrix would leave the second kernel none)
  auto apart = [&](const double* x, int len) { return x + len <= a || a + p * p <= x; };
  const bool near = p >= kNearMinP && apart(evals, p) && apart(evecs, p * p);
  if (near || p <= 2)
    hipLaunchKernelGGL(k_small_eigh_near, dim3(1), dim3(1024), kEigLdsBytes, s, a, p, evals, evecs, sweeps);
  if (near)
    hipLaunchKernelGGL(k_small_eigh<true>, dim3(1), dim3(kEigThreads), kEigLdsBytes, s, a, p, evals, evecs, sweeps);
  else if (p > 2)
    hipLaunchKernelGGL(k_small_eigh<false>, dim3(1), dim3(kEigThreads), kEigLdsBytes, s, a, p, evals, evecs, sweeps);
  return hipGetLastError();
}

}  // namespace lobpcg
