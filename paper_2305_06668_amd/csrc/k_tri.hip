// Tridiagonal preconditioner (Sec. 4.4, Table 1: the diagonal plus the upper
// and lower diagonal elements of A, where the paper solves with LAPACK's
// Gaussian elimination).  Column j of R (n x nact, row-major, leading
// dimension ld) is replaced in place by the solution w of T_j w = r with
//   T_j = tridiag(e, t, e),  t_i = max(|d_i - theta_j|, |e_{i-1}| + |e_i| + delta_j),
// e_i = a_{i,i+1}, d = diag(A), delta_j = kPrecondGuard max(1, |theta_j|):
// symmetric and strictly diagonally dominant with a positive diagonal, so
// elimination without pivoting is stable.
//
// Partition method.  A run of rows is described by its interface, its first
// and last unknowns as affine functions of the two just outside it,
//   x_first = ys + vs x_left + ws x_right,  x_last = ye + ve x_left + we x_right,
// and the interfaces of two neighbouring runs give the one of both (Iface,
// merge).  A thread takes a chunk of L rows of one column, a workgroup a group
// of 256 / CW neighbouring chunks:
//   k_tri_rows<false>  a UL and an LU sweep over the chunk give its interface;
//                      the chunks' are merged to the group's (across lanes,
//                      then across the waves through LDS);
//   k_tri_top          workgroup j: the groups' interfaces are merged up a tree
//                      in LDS, the values beside each group come down again;
//   k_tri_rows<true>   the same sweeps, with the factors kept in registers;
//                      the values beside the group come down the same merges
//                      to each chunk, which is then solved in registers.
// Every sum and factor is fp64, whatever R holds.
//
// R is read twice and written once (n = 1e6, 16 columns: 384 MB, part of the
// second read from the last-level cache): 47 + 10 + 67 us there, bound by the
// rows' loads and the sweeps behind them, which overlap only across the two to
// four workgroups of a CU.  With 1024 chunks of 977 rows the sweeps were 16 k
// serial chains of divisions over strided rows, R passed memory five times and
// one thread per column ran through the 1024 chunks: 400 + 210 + 420 us.
#include <algorithm>

#include "internal.h"

namespace lobpcg {

namespace {

typedef double dd2 __attribute__((ext_vector_type(2)));

struct Iface {
  double ys, vs, ws, ye, ve, we;
};

// The unknowns a (last of the left run) and b (first of the right run) at the
// seam of two runs, as functions of the unknowns outside both.
struct Seam {
  double a0, al, ar, b0, bl, br;
};

// 1 / q (q > 0) to 1 ulp: the hardware estimate and two Newton steps; 0 for an
// infinite pivot, as a division gives it: a row whose diagonal entry is infinite
// is frozen at 0 and its neighbours do not couple through it.  (There the
// estimate is 0 and stays so, as the steps' q is finite, which costs nothing
// beside the estimate; a fix-up behind the steps is 1 % of the whole solve.)
__device__ __forceinline__ double rcp2(double q) {
  double r = __builtin_amdgcn_rcp(q);
  const double f = fmin(q, 0x1.fffffffffffffp+1023);
  r = fma(r, fma(-f, r, 1.0), r);
  return fma(r, fma(-f, r, 1.0), r);
}

// A, B: neighbouring runs; returns the interface of both
__device__ __forceinline__ Iface merge(const Iface& A, const Iface& B, Seam& s) {
  const double k = rcp2(fma(-A.we, B.vs, 1.0));
  s.a0 = fma(A.we, B.ys, A.ye) * k;
  s.al = A.ve * k;
  s.ar = A.we * B.ws * k;
  s.b0 = fma(B.vs, s.a0, B.ys);
  s.bl = B.vs * s.al;
  s.br = fma(B.vs, s.ar, B.ws);
  Iface o;
  o.ys = fma(A.ws, s.b0, A.ys);
  o.vs = fma(A.ws, s.bl, A.vs);
  o.ws = A.ws * s.br;
  o.ye = fma(B.ve, s.a0, B.ye);
  o.ve = B.ve * s.al;
  o.we = fma(B.ve, s.ar, B.we);
  return o;
}

// the values (left, right) outside a pair of runs become those outside one of
// them: the right run's when `right`, else the left one's
__device__ __forceinline__ void descend(const Seam& s, bool right, double& xl, double& xr) {
  const double a = fma(s.ar, xr, fma(s.al, xl, s.a0));
  const double b = fma(s.br, xr, fma(s.bl, xl, s.b0));
  if (right) xl = a;
  else xr = b;
}

// the lower and the upper lane's value of the pair (lane, lane ^ M)
template <int M>
__device__ __forceinline__ void lane_pair(double v, bool upper, double& lo, double& hi) {
  if constexpr (M == 16 || M == 32) {
    const auto l = (M == 16) ? __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false)
                             : __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = (M == 16) ? __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false)
                             : __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    lo = __hiloint2double(h[0], l[0]);
    hi = __hiloint2double(h[1], l[1]);
  } else {
    const double o = __shfl_xor(v, M);
    lo = upper ? o : v;
    hi = upper ? v : o;
  }
}
template <int M>
__device__ __forceinline__ Iface merge_lanes(const Iface& f, bool upper, Seam& s) {
  Iface A, B;
  lane_pair<M>(f.ys, upper, A.ys, B.ys);
  lane_pair<M>(f.vs, upper, A.vs, B.vs);
  lane_pair<M>(f.ws, upper, A.ws, B.ws);
  lane_pair<M>(f.ye, upper, A.ye, B.ye);
  lane_pair<M>(f.ve, upper, A.ve, B.ve);
  lane_pair<M>(f.we, upper, A.we, B.we);
  return merge(A, B, s);
}

// L rows per chunk, CW columns side by side (nact of them real).  Rows past n
// continue the system by uncoupled rows with r = 0.
template <typename T, int L, int CW, bool SOLVE>
__global__ __launch_bounds__(256, SOLVE ? 2 : 4) void k_tri_rows(T* R, int64_t ld, int nact, int64_t n,
                                                  const double* __restrict__ theta,
                                                  const double* __restrict__ d,
                                                  const double* __restrict__ e,
                                                  const double* __restrict__ off,
                                                  double* __restrict__ bnd,
                                                  const double* __restrict__ xb) {
  constexpr int NQ = 256 / CW;  // chunks per group
  constexpr int LP = L + 1;
  __shared__ dd2 sdo[NQ * LP];      // (d, off) of row u of chunk q at q LP + u (a stride off the banks)
  __shared__ double se[NQ * LP];    // the coupling of that row to the one above; u = L: below the last
  __shared__ Iface wf[4][CW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = blockIdx.y * CW + (tid & (CW - 1)), q = tid / CW;
  const int64_t g = blockIdx.x, r0 = g * (NQ * L);
  const bool live = j < nact;
  const int64_t row = r0 + (int64_t)q * L;
  T* Rj = R + row * ld + (live ? j : 0);
  double x[L];
#pragma unroll
  for (int u = 0; u < L; ++u) x[u] = (live && row + u < n) ? (double)Rj[u * ld] : 0.0;
  const double th = live ? theta[j] : 0.0;
  const double delta = kPrecondGuard * fmax(1.0, fabs(th));
  for (int i = tid; i < NQ * L; i += 256) {
    const int64_t r = r0 + i;
    const int qq = i / L, at = qq * LP + (i - qq * L);
    sdo[at] = (r < n) ? dd2{d[r], off[r]} : dd2{0.0, 1.0};
    const double ei = (r > 0 && r <= n) ? e[r - 1] : 0.0;  // (e[n - 1] = 0)
    se[at] = ei;
    if (i == qq * L && qq > 0) se[qq * LP - 1] = ei;
  }
  if (tid == 0) {
    const int64_t r = r0 + NQ * L;
    se[NQ * LP - 1] = (r <= n) ? e[r - 1] : 0.0;
  }
  __syncthreads();
  const dd2* cdo = sdo + q * LP;
  const double* ce = se + q * LP;
  const double a_s = ce[0], c_e = ce[L];
  auto diag = [&](int u) {
    const dd2 t = cdo[u];
    return fmax(fabs(t[0] - th), t[1] + delta);
  };
  Iface f;
  {
    // UL sweep up: the first row
    double ap = 0.0, sy = 0.0, sw = 0.0, inv = 1.0;
#pragma unroll
    for (int u = L - 1; u >= 0; --u) {
      const double ec = (u == L - 1) ? 0.0 : ce[u + 1];
      inv = rcp2(fma(-ec, ap, diag(u)));
      sy = fma(-ec, sy, x[u]) * inv;
      sw = ((u == L - 1) ? -c_e : -ec * sw) * inv;
      ap = ce[u] * inv;
    }
    f.ys = sy;
    f.vs = -a_s * inv;
    f.ws = sw;
  }
  // (the diagonal and the couplings are read again: kept in registers they
  // would cost two of four waves per SIMD)
  asm volatile("" ::: "memory");
  double iv[SOLVE ? L : 1];
  {
    // LU sweep down: the last row; SOLVE keeps the pivots' reciprocals and
    // leaves the forward right-hand side in x
    double cp = 0.0, ry = 0.0, rv = 0.0, inv = 1.0;
#pragma unroll
    for (int u = 0; u < L; ++u) {
      const double ea = (u == 0) ? 0.0 : ce[u];
      inv = rcp2(fma(-ea, cp, diag(u)));
      ry = fma(-ea, ry, x[u]) * inv;
      rv = ((u == 0) ? -a_s : -ea * rv) * inv;
      cp = ce[u + 1] * inv;
      if (SOLVE) {
        iv[u] = inv;
        x[u] = ry;
      }
    }
    f.ye = ry;
    f.ve = rv;
    f.we = -c_e * inv;
  }
  // merge the wave's chunks, then the waves'
  Seam s4, s8, s16, s32, w01, w23, top;
  if constexpr (CW <= 4) f = merge_lanes<4>(f, (lane & 4) != 0, s4);
  if constexpr (CW <= 8) f = merge_lanes<8>(f, (lane & 8) != 0, s8);
  f = merge_lanes<16>(f, (lane & 16) != 0, s16);
  f = merge_lanes<32>(f, (lane & 32) != 0, s32);
  if (lane < CW) wf[wave][lane] = f;
  __syncthreads();
  const int c = tid & (CW - 1);
  const Iface f01 = merge(wf[0][c], wf[1][c], w01), f23 = merge(wf[2][c], wf[3][c], w23);
  f = merge(f01, f23, top);
  if constexpr (!SOLVE) {
    if (tid < CW && live) {
      // one run of groups per column and coefficient, as k_tri_top reads them
      const int64_t P = gridDim.x;
      double* o = bnd + (int64_t)j * 6 * P + g;
      o[0] = f.ys;
      o[P] = f.vs;
      o[2 * P] = f.ws;
      o[3 * P] = f.ye;
      o[4 * P] = f.ve;
      o[5 * P] = f.we;
    }
  } else {
    // down again to the values beside this chunk
    const double* xj = xb + (int64_t)j * 2 * gridDim.x + g;
    double xl = live ? xj[0] : 0.0;
    double xr = live ? xj[gridDim.x] : 0.0;
    descend(top, wave >= 2, xl, xr);
    if (wave >= 2) descend(w23, wave == 3, xl, xr);
    else descend(w01, wave == 1, xl, xr);
    descend(s32, (lane & 32) != 0, xl, xr);
    descend(s16, (lane & 16) != 0, xl, xr);
    if constexpr (CW <= 8) descend(s8, (lane & 8) != 0, xl, xr);
    if constexpr (CW <= 4) descend(s4, (lane & 4) != 0, xl, xr);
    // forward right-hand side with the left neighbour, then back
    double t = xl;
#pragma unroll
    for (int u = 0; u < L; ++u) {
      t *= -ce[u] * iv[u];
      x[u] += t;
    }
    double y = xr;
#pragma unroll
    for (int u = L - 1; u >= 0; --u) {
      y = fma(-ce[u + 1] * iv[u], y, x[u]);
      x[u] = y;
    }
#pragma unroll
    for (int u = 0; u < L; ++u)
      if (live && row + u < n) Rj[u * ld] = (T)x[u];
  }
}

// One workgroup per column: P groups' interfaces (bnd) -> the values left and
// right of each group (xb).  Thread t takes `per` neighbouring groups (one up
// to 1024 of them), merged in order; the threads' interfaces go up a binary
// tree in LDS (level of node i in [NP, 2 NP) the leaves, i / 2 its parent) and
// the outside values down it.
constexpr int kTopThreads = 1024;
__global__ __launch_bounds__(kTopThreads) void k_tri_top(int64_t P, int per, int NP,
                                                         double* __restrict__ bnd,
                                                         double* __restrict__ xb) {
  extern __shared__ __attribute__((aligned(16))) char top_smem[];
  Iface* node = reinterpret_cast<Iface*>(top_smem);  // 2 NP (index 0 unused)
  dd2* out = reinterpret_cast<dd2*>(node + 2 * NP);  // (left, right) of each node
  const int j = blockIdx.x, t = threadIdx.x;
  const int64_t g0 = (int64_t)t * per, g1 = min(P, g0 + per);
  bnd += (int64_t)j * 6 * P;
  xb += (int64_t)j * 2 * P;
  auto load = [&](int64_t g) {
    return Iface{bnd[g], bnd[P + g], bnd[2 * P + g], bnd[3 * P + g], bnd[4 * P + g], bnd[5 * P + g]};
  };
  // the thread's run; the last-row part of each prefix replaces the group's own
  Iface f{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (g0 < g1) f = load(g0);
  for (int64_t g = g0 + 1; g < g1; ++g) {
    Seam s;
    f = merge(f, load(g), s);
    bnd[3 * P + g] = f.ye;
    bnd[4 * P + g] = f.ve;
    bnd[5 * P + g] = f.we;
  }
  if (t < NP) node[NP + t] = f;
  __syncthreads();
  for (int w = NP >> 1; w >= 1; w >>= 1) {
    if (t < w) {
      Seam s;
      node[w + t] = merge(node[2 * (w + t)], node[2 * (w + t) + 1], s);
    }
    __syncthreads();
  }
  if (t == 0) out[1] = dd2{0.0, 0.0};
  __syncthreads();
  for (int w = 1; w < NP; w <<= 1) {
    if (t < w) {
      const int i = w + t;
      Seam s;
      merge(node[2 * i], node[2 * i + 1], s);
      const dd2 o = out[i];
      double l0 = o[0], r0 = o[1], l1 = o[0], r1 = o[1];
      descend(s, false, l0, r0);
      descend(s, true, l1, r1);
      out[2 * i] = dd2{l0, r0};
      out[2 * i + 1] = dd2{l1, r1};
    }
    __syncthreads();
  }
  if (g0 >= g1) return;
  // back through the thread's run: group g's left value is the last unknown of
  // the prefix before it, whose right value is group g's first unknown
  const dd2 o = out[NP + t];
  double right = o[1];
  for (int64_t g = g1 - 1; g >= g0; --g) {
    double left = o[0], first = 0.0;
    if (g > g0) {
      const double ys = bnd[g], vs = bnd[P + g], ws = bnd[2 * P + g];  // own first row
      const double ye = bnd[3 * P + g - 1], ve = bnd[4 * P + g - 1], we = bnd[5 * P + g - 1];  // prefix's last
      const double pa = fma(ve, o[0], ye);     // last of the prefix without `first`
      const double fb = fma(ws, right, ys);    // first of g without `left`
      left = fma(we, fb, pa) * rcp2(fma(-we, vs, 1.0));
      first = fma(vs, left, fb);
    }
    xb[g] = left;
    xb[P + g] = right;
    right = first;
  }
}

constexpr int kTriNarrow = 16, kTriWide = 32;  // rows per chunk

template <typename T, int L, int CW>
hipError_t tri_launch(T* R, int64_t ld, int nact, int64_t n, const double* theta, const double* d,
                      const double* e, const double* off, double* bnd, double* xb, hipStream_t s) {
  const int64_t P = (n + (256 / CW) * L - 1) / ((256 / CW) * L);
  const dim3 grid((unsigned)P, (unsigned)((nact + CW - 1) / CW));
  hipLaunchKernelGGL((k_tri_rows<T, L, CW, false>), grid, dim3(256), 0, s, R, ld, nact, n, theta, d, e, off, bnd,
                     xb);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  static bool attr = false;
  if (!attr) {
    err = hipFuncSetAttribute(reinterpret_cast<const void*>(k_tri_top), hipFuncAttributeMaxDynamicSharedMemorySize,
                              2 * kTopThreads * (int)(sizeof(Iface) + sizeof(dd2)));
    if (err != hipSuccess) return err;
    attr = true;
  }
  const int per = (int)((P + kTopThreads - 1) / kTopThreads);
  int NP = 1;
  while (NP * (int64_t)per < P) NP <<= 1;
  hipLaunchKernelGGL(k_tri_top, dim3(nact), dim3(std::max(64, NP)), 2 * NP * (sizeof(Iface) + sizeof(dd2)), s, P,
                     per, NP, bnd, xb);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((k_tri_rows<T, L, CW, true>), grid, dim3(256), 0, s, R, ld, nact, n, theta, d, e, off, bnd,
                     xb);
  return hipGetLastError();
}

// Chunks of 32 rows where they fill the chip (two waves per SIMD), of 16 below
// that: half the length of every chain.  Columns in blocks of 16, 8 or 4.
template <typename T, int CW>
hipError_t tri_rows(T* R, int64_t ld, int nact, int64_t n, const double* theta, const double* d,
                    const double* e, const double* off, double* bnd, double* xb, hipStream_t s) {
  const int64_t threads = n / kTriWide * ((nact + CW - 1) / CW * CW);
  return threads >= 2 * 1024 * 64
             ? tri_launch<T, kTriWide, CW>(R, ld, nact, n, theta, d, e, off, bnd, xb, s)
             : tri_launch<T, kTriNarrow, CW>(R, ld, nact, n, theta, d, e, off, bnd, xb, s);
}

template <typename T>
hipError_t tri_apply_any(T* R, int64_t ld, int nact, int64_t n, const double* theta, const double* d,
                         const double* e, const double* off, double* bnd, double* xb, double* scr,
                         hipStream_t s) {
  if (n < 1 || nact < 1 || nact > 64 || ld < nact) return hipErrorInvalidValue;
  if (tri_scratch(n, nact) > 0) {
    bnd = scr;
    xb = scr + (n / 256 + 1) * 6 * nact;
  }
  if (nact <= 4) return tri_rows<T, 4>(R, ld, nact, n, theta, d, e, off, bnd, xb, s);
  if (nact <= 8) return tri_rows<T, 8>(R, ld, nact, n, theta, d, e, off, bnd, xb, s);
  return tri_rows<T, 16>(R, ld, nact, n, theta, d, e, off, bnd, xb, s);
}

}  // namespace

hipError_t tri_apply_f64(double* R, int64_t ld, int nact, int64_t n, const double* theta,
                         const double* d, const double* e, const double* off, double* bnd,
                         double* xb, double* scr, hipStream_t s) {
  return tri_apply_any<double>(R, ld, nact, n, theta, d, e, off, bnd, xb, scr, s);
}
hipError_t tri_apply_f32(float* R, int64_t ld, int nact, int64_t n, const double* theta,
                         const double* d, const double* e, const double* off, double* bnd,
                         double* xb, double* scr, hipStream_t s) {
  return tri_apply_any<float>(R, ld, nact, n, theta, d, e, off, bnd, xb, scr, s);
}

// ---- the off-diagonal e_i = a_{i,i+1} and off_i = |e_{i-1}| + |e_i| ------

__global__ void k_tri_off_csr(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                              const double* __restrict__ val, int64_t n, double* __restrict__ e) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double v = 0.0;
  for (int k = rp[i]; k < rp[i + 1]; ++k)
    if ((int64_t)ci[k] == i + 1) v += val[k];
  e[i] = v;
}

__global__ void k_tri_off_dense(const double* __restrict__ A, int64_t lda, int64_t n,
                                double* __restrict__ e) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  e[i] = (i + 1 < n) ? A[i * lda + i + 1] : 0.0;
}

// H = A (x) I + I (x) A + diag(vec V): entry (i na + j, i na + j + 1) is
// A[j][j+1] inside a block of na rows, 0 across blocks
__global__ void k_tri_off_kron(const double* __restrict__ A, int64_t na, double* __restrict__ e) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= na * na) return;
  const int64_t j = r % na;
  e[r] = (j + 1 < na) ? A[j * na + j + 1] : 0.0;
}

__global__ void k_tri_rowoff(const double* __restrict__ e, int64_t n, double* __restrict__ off) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  off[i] = fabs(e[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0);
}

static hipError_t rowoff(const double* e, int64_t n, double* off, hipStream_t s) {
  hipLaunchKernelGGL(k_tri_rowoff, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, e, n, off);
  return hipGetLastError();
}

hipError_t tri_offdiag_csr(const int32_t* rp, const int32_t* ci, const double* val, int64_t n,
                           double* e, double* off, hipStream_t s) {
  hipLaunchKernelGGL(k_tri_off_csr, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rp, ci, val, n,
                     e);
  hipError_t err = hipGetLastError();
  return err != hipSuccess ? err : rowoff(e, n, off, s);
}
hipError_t tri_offdiag_dense(const double* A, int64_t lda, int64_t n, double* e, double* off,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_tri_off_dense, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, A, lda, n,
                     e);
  hipError_t err = hipGetLastError();
  return err != hipSuccess ? err : rowoff(e, n, off, s);
}
hipError_t tri_offdiag_kron(const double* A, int64_t na, double* e, double* off, hipStream_t s) {
  const int64_t n = na * na;
  hipLaunchKernelGGL(k_tri_off_kron, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, A, na, e);
  hipError_t err = hipGetLastError();
  return err != hipSuccess ? err : rowoff(e, n, off, s);
}

}  // namespace lobpcg
