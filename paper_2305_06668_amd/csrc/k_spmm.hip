// CSR SpMM Y = A W (Alg. 1: the products A X^[0] and A W^[k] for a sparse
// operator).  The (col, val) stream is read from HBM once; every stored entry
// then needs one row of W (ncols * s contiguous bytes), gathered through L2.
// For the banded workloads the W window stays in L2 (hit rate ~90 %, HBM
// traffic within 1 % of the algorithmic bytes).  Three kernels:
//   * k_spmm_block and k_spmm_rows (2 fp64 / 4 fp32 columns per lane, 16-byte
//     loads; a workgroup, or each wave for itself, stages its rows' (col, val)
//     range in LDS): the fewest instructions and wave slots per gathered row,
//     used from 5 (fp64) or 9 (fp32) columns;
//   * k_spmm_csr (one column per lane, (col, val) broadcast by shuffles):
//     narrow blocks, and some misaligned ones (see spmm_any).
// Row blocks are remapped so that each XCD (hardware dispatches block b to
// XCD b % 8) walks one contiguous range of rows: a banded matrix then keeps
// its W window inside that XCD's L2.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"

namespace lobpcg {

// G = lanes per stored entry (1, 2, 4, 8 or 16 >= ncols); a row is owned by a group
// of 16 lanes, which holds NP = 16 / G "slots" that take stored entries in turn.
// The group loads its row's (col, val) pairs in chunks of 16 (one per lane,
// coalesced), two or four chunks up front, broadcasts them with __shfl, and issues
// all gathers of a pass (G >= 8: of a chunk) before accumulating.  Slot partial
// sums are combined with xor shuffles at the end.
template <typename TV, typename TW, int G>
__global__ __launch_bounds__(256) void k_spmm_csr(const int32_t* __restrict__ rp,
                                                  const int32_t* __restrict__ ci,
                                                  const TV* __restrict__ val,
                                                  const TW* __restrict__ W, int64_t ldw,
                                                  TW* __restrict__ Y, int64_t ldy, int ncols,
                                                  int64_t n, int per_xcd) {
  constexpr int GS = 16;
  constexpr int NP = GS / G;
  constexpr int RPB = 256 / GS;
  // narrow blocks (G <= 2) take four chunks per pass: a row's entries then
  // fit one pass, and every gather of the pass is in flight together
  constexpr int NCH = (G <= 2) ? 4 : 2;
  const int b = blockIdx.x;
  const int lb = (b & 7) * per_xcd + (b >> 3);
  const int64_t row = (int64_t)lb * RPB + threadIdx.x / GS;
  const int lg = threadIdx.x & (GS - 1);
  const int slot = lg / G;
  const int c = lg & (G - 1);
  const int gbase = (threadIdx.x & 63) & ~(GS - 1);
  if (row >= n) return;  // the whole group shares the row
  const bool active = c < ncols;
  const int e0 = rp[row], e1 = rp[row + 1];
  TW acc = TW(0);
  for (int e = e0; e < e1; e += NCH * GS) {
    int colr[NCH];
    TV vr[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int ee = e + k * GS + lg;
      const bool ok = ee < e1;
      colr[k] = ok ? ci[ee] : 0;
      vr[k] = ok ? val[ee] : TV(0);
    }
    if constexpr (G <= 4) {
      // all gathers of the pass first, then the products in the same order
      // as below (entries past the row end contribute 0 * 0)
      TW w[NCH][G];
      TV vv[NCH][G];
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int base_e = e + k * GS;
#pragma unroll
        for (int u = 0; u < G; ++u) {
          const int t = slot + NP * u;
          const int cidx = __shfl(colr[k], gbase + t, 64);
          vv[k][u] = __shfl(vr[k], gbase + t, 64);
          w[k][u] = (active && base_e + t < e1) ? W[(int64_t)cidx * ldw + c] : TW(0);
        }
      }
#pragma unroll
      for (int k = 0; k < NCH; ++k)
#pragma unroll
        for (int u = 0; u < G; ++u) acc += (TW)vv[k][u] * w[k][u];
      continue;
    }
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int base_e = e + k * GS;
      if (base_e >= e1) break;
      TW w[G];
      TV vv[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int t = slot + NP * u;
        const int cidx = __shfl(colr[k], gbase + t, 64);
        vv[u] = __shfl(vr[k], gbase + t, 64);
        w[u] = (active && base_e + t < e1) ? W[(int64_t)cidx * ldw + c] : TW(0);
      }
#pragma unroll
      for (int u = 0; u < G; ++u) acc += (TW)vv[u] * w[u];
    }
  }
#pragma unroll
  for (int off = G; off < GS; off <<= 1) acc += __shfl_xor(acc, off, 64);
  if (slot == 0 && active) Y[row * ldy + c] = acc;
}

template <typename TV, typename TW, int G>
static hipError_t spmm_launch(const int32_t* rp, const int32_t* ci, const TV* val, const TW* W,
                              int64_t ldw, TW* Y, int64_t ldy, int ncols, int64_t n,
                              hipStream_t s) {
  constexpr int RPB = 256 / 16;
  const int64_t nb = (n + RPB - 1) / RPB;
  const int64_t nbp = (nb + 7) / 8 * 8;
  hipLaunchKernelGGL((k_spmm_csr<TV, TW, G>), dim3((unsigned)nbp), dim3(256), 0, s, rp, ci, val,
                     W, ldw, Y, ldy, ncols, n, (int)(nbp / 8));
  return hipGetLastError();
}


// 16 bytes of CPL elements at element alignment (a global load of four dwords
// needs no more than a dword's)
template <typename T, int CPL>
struct Vec16;
template <>
struct Vec16<double, 2> {
  typedef double __attribute__((ext_vector_type(2), aligned(8))) type;
};
template <>
struct Vec16<float, 4> {
  typedef float __attribute__((ext_vector_type(4), aligned(4))) type;
};

// a stored entry in LDS: where its W row starts and its value, one LDS read
template <typename TW> struct Entry;
template <> struct alignas(16) Entry<double> { uint32_t at; uint32_t pad; double v; };
template <> struct alignas(8) Entry<float> { uint32_t at; float v; };

// Sum of m staged entries times their W rows, added to acc in order, four
// gathers in flight; only what is stored is gathered or multiplied.
template <int CPL, typename TW, typename VT, class Gather>
__device__ __forceinline__ void add_entries(const Entry<TW>* x, int m, VT& acc, Gather&& gather) {
  constexpr int UN = 4;
  int t = 0;
  for (; t + UN <= m; t += UN) {
    VT w[UN];
    TW v[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const Entry<TW> en = x[t + u];
      v[u] = en.v;
      w[u] = gather(en);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int q = 0; q < CPL; ++q) acc[q] += v[u] * w[u][q];
  }
  if (t < m) {
    VT w[UN - 1];
    TW v[UN - 1];
#pragma unroll
    for (int u = 0; u < UN - 1; ++u) {
#pragma unroll
      for (int q = 0; q < CPL; ++q) w[u][q] = TW(0);
      v[u] = TW(0);
      if (t + u < m) {
        const Entry<TW> en = x[t + u];
        v[u] = en.v;
        w[u] = gather(en);
      }
    }
#pragma unroll
    for (int u = 0; u < UN - 1; ++u)
      if (t + u < m) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[q] += v[u] * w[u][q];
      }
  }
}
template <bool NT, typename T>
__device__ __forceinline__ T stream_load(const T* p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}

// In both kernels G lanes take a row; lane l of them holds columns c .. c +
// CPL - 1, c = min(l CPL, ncols - CPL) (the last lanes may repeat columns, so
// that every load is whole), and gathers them with one 16-byte load per stored
// entry.  Entries are accumulated in CSR order.
// BIG: W spans 4 GB or more, LDS holds the column and the address is formed in
// 64 bits; else it holds the byte offset, added to a scalar base by the load.
// NT: the matrix is read with the non-temporal hint (see spmm_stream_launch).
// What bounds them: a 16-byte load of 64 lanes takes the L1 16 cycles, hit or
// not, so every gather that is issued for a lane group whose row has ended is
// lost (rows of 41 +- 4.5 entries, eight to a wave: 55 issued with eight in
// flight, 49 with four), and loads return in order, so the gathers behind a
// fetch of entries wait for HBM.  Gathers alone take 160 us for the n = 1e6,
// 41 entries per row, 16-column fp64 product, the entries alone 125 us, both
// together without rows or sums 230 to 270 us; the product takes 355.

// k_spmm_block: a workgroup takes 256 / G consecutive rows and copies their
// range of entries to LDS (coalesced), `cap` entries at a time (block_lds),
// between barriers; nothing is in flight across them, but six to eight
// workgroups share a CU.
template <typename TV, typename TW, int G, int CPL, bool BIG, bool NT>
__global__ __launch_bounds__(256) void k_spmm_block(const int32_t* __restrict__ rp,
                                                    const int32_t* __restrict__ ci,
                                                    const TV* __restrict__ val,
                                                    const TW* __restrict__ W, int64_t ldw,
                                                    TW* __restrict__ Y, int64_t ldy, int ncols,
                                                    int64_t n, int per_xcd, unsigned cap) {
  typedef typename Vec16<TW, CPL>::type VT;
  constexpr int RPB = 256 / G;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  Entry<TW>* E = reinterpret_cast<Entry<TW>*>(lds);
  const int b = blockIdx.x;
  const int lb = (b & 7) * per_xcd + (b >> 3);
  const int64_t r0 = (int64_t)lb * RPB;
  if (r0 >= n) return;  // whole block
  const int l = threadIdx.x % G;
  const int64_t row = r0 + threadIdx.x / G;
  const int c = min(l * CPL, ncols - CPL);
  const uint32_t rowb = (uint32_t)(ldw * sizeof(TW)), cb = (uint32_t)(c * sizeof(TW));
  const TW* Wc = W + c;
  const int B0 = rp[r0];
  const unsigned total = (unsigned)(rp[min(r0 + RPB, n)] - B0);
  const unsigned e0 = (unsigned)(rp[min(row, n)] - B0), e1 = (unsigned)(rp[min(row + 1, n)] - B0);
  auto gather = [&](const Entry<TW>& x) {
    if (BIG) return *reinterpret_cast<const VT*>(Wc + (int64_t)x.at * ldw);
    return *reinterpret_cast<const VT*>(reinterpret_cast<const char*>(W) + (x.at + cb));
  };
  VT acc;
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q] = TW(0);
  for (unsigned p = 0; p < total; p += cap) {
    const unsigned cnt = min(cap, total - p);
    const int32_t* cp = ci + B0 + (int64_t)p;
    const TV* vp = val + B0 + (int64_t)p;
    __syncthreads();  // the previous pass is consumed
    for (unsigned i = threadIdx.x; i < cnt; i += 256) {
      const uint32_t col = (uint32_t)stream_load<NT>(cp + i);
      Entry<TW> x;
      x.at = BIG ? col : col * rowb;
      x.v = (TW)stream_load<NT>(vp + i);
      E[i] = x;
    }
    __syncthreads();
    const unsigned a = max(e0, p), z = min(e1, p + cnt);
    if (a < z) add_entries<CPL>(E + (a - p), (int)(z - a), acc, gather);
  }
  if (row < n && l * CPL < ncols) *reinterpret_cast<VT*>(Y + row * ldy + c) = acc;
}

// k_spmm_rows: a wave takes 64 / G consecutive rows at a time and copies their
// range of entries (coalesced) to its own part of LDS.  Everything is private
// to the wave (no barrier), waves walk on through their XCD's rows, and while a
// wave gathers for one group of rows its loads of the next group's entries and
// of the row pointers after that are in flight.  The groups whose entries do not
// fit (kRowCap per row on average) are passed over and taken by themselves after
// every 64 groups, in passes of up to kRowPass entries of every row, each pass's
// loads in flight during the one before it.  (With both kinds in one loop the
// compiler waits for the loads of one where it goes on with the other: rows that
// all fit took 3 to 15 % longer.)
constexpr int kRowCap = 48, kRowPass = 44;
constexpr int64_t kCacheBytes = 280000000;  // the memory-side cache, 268, and a little that passes
constexpr int kRowsWaves(int G) { return G == 4 ? 3 : 4; }  // workgroups per CU: their registers and LDS
template <typename TV, typename TW, int G, int CPL, bool BIG, bool NT>
__global__ __launch_bounds__(256)
void k_spmm_rows(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                 const TV* __restrict__ val, const TW* __restrict__ W, int64_t ldw,
                 TW* __restrict__ Y, int64_t ldy, int ncols, int64_t n, int per_xcd) {
  typedef typename Vec16<TW, CPL>::type VT;
  constexpr int NR = 64 / G;             // rows per wave and step
  constexpr int CAP = kRowCap * NR;      // entries in the wave's LDS
  constexpr int NL = CAP / 64;           // entries per lane and copy
  constexpr int NQ = (kRowPass + G - 1) / G;  // ... and pass by rows
  __shared__ Entry<TW> lds[4][CAP];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Entry<TW>* E = lds[wave];
  const int r = lane / G, l = lane % G;
  const int c = min(l * CPL, ncols - CPL);
  const uint32_t rowb = (uint32_t)(ldw * sizeof(TW)), cb = (uint32_t)(c * sizeof(TW));
  const TW* Wc = W + c;
  // this wave's groups of rows: first, first + step, ... below last
  const int64_t first = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3) * 4 + wave;
  const int step = (gridDim.x >> 3) * 4;
  const int64_t last = min((int64_t)((blockIdx.x & 7) + 1) * per_xcd, (n + NR - 1) / NR);
  if (first >= last) return;
  // row pointers of this lane's row of group g (empty past the matrix)
  auto load_rp = [&](int64_t g, int& e0, int& e1) {
    const int64_t row = min(g * NR + r, n);
    e0 = rp[row];
    e1 = rp[min(row + 1, n)];
  };
  // the group's range of entries: the first row's start, the last row's end
  auto lo_of = [&](int e0) { return __builtin_amdgcn_readlane(e0, 0); };
  auto hi_of = [&](int e1) { return __builtin_amdgcn_readlane(e1, 63); };
  // entries first + stride k below cnt, counted from cp and vp, into registers
  auto fetch = [&](auto& pc, auto& pv, const int32_t* cp, const TV* vp, int first, auto stride, int cnt) {
#pragma unroll
    for (int k = 0; k < (int)(sizeof(pc) / sizeof(pc[0])); ++k) {
      const int i = first + stride() * k;
      if (i < cnt) {
        pc[k] = stream_load<NT>(cp + i);
        pv[k] = stream_load<NT>(vp + i);
      }
    }
  };
  // and from there to x
  auto stage = [&](const auto& pc, const auto& pv, Entry<TW>* x, int first, auto stride, int cnt) {
#pragma unroll
    for (int k = 0; k < (int)(sizeof(pc) / sizeof(pc[0])); ++k) {
      const int i = first + stride() * k;
      if (i < cnt) {
        Entry<TW> en;
        en.at = BIG ? (uint32_t)pc[k] : (uint32_t)pc[k] * rowb;
        en.v = (TW)pv[k];
        x[i] = en;
      }
    }
  };
  auto lds_ready = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const std::integral_constant<int, 64> flat{};
  const std::integral_constant<int, G> by_row{};
  auto gather = [&](const Entry<TW>& x) {
    if (BIG) return *reinterpret_cast<const VT*>(Wc + (int64_t)x.at * ldw);
    return *reinterpret_cast<const VT*>(reinterpret_cast<const char*>(W) + (x.at + cb));
  };
  auto zero = [&]() {
    VT a;
#pragma unroll
    for (int q = 0; q < CPL; ++q) a[q] = TW(0);
    return a;
  };
  auto store = [&](int64_t g, const VT& acc) {
    const int64_t row = g * NR + r;
    if (row < n && l * CPL < ncols) *reinterpret_cast<VT*>(Y + row * ldy + c) = acc;
  };
  for (int64_t base = first; base < last; base += (int64_t)64 * step) {
    const int64_t stop = min(last, base + (int64_t)64 * step);
    uint64_t rest = 0;  // the groups that do not fit
    int e0, e1, f0, f1;  // row pointers of this group and the next
    {
      load_rp(base, e0, e1);
      load_rp(base + step, f0, f1);
      int b0 = lo_of(e0), cnt = hi_of(e1) - b0;
      int32_t pc[NL];
      TV pv[NL];
      if (cnt <= CAP) fetch(pc, pv, ci + b0, val + b0, lane, flat, cnt);
      uint64_t bit = 1;
      for (int64_t g = base; g < stop; g += step, bit <<= 1) {
        const bool fits = cnt <= CAP;
        // (the previous group's gathers have returned: their LDS reads are done)
        if (fits) stage(pc, pv, E, lane, flat, cnt);
        // the next group's entries and the row pointers of the one after it
        const int nb0 = lo_of(f0), ncnt = hi_of(f1) - nb0;
        if (g + step < stop && ncnt <= CAP) fetch(pc, pv, ci + nb0, val + nb0, lane, flat, ncnt);
        int g0, g1;
        load_rp(g + 2 * step, g0, g1);
        // vmcnt(0): loads return in order, so the gathers would wait for these in
        // any case, with fewer of the waves' gathers in each other's way so (fp32,
        // 16 columns: 246 -> 233 us; fp64, 8: 253 -> 244, 16: 322 -> 315)
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if (fits) {
          VT acc = zero();
          lds_ready();
          add_entries<CPL>(E + (e0 - b0), e1 - e0, acc, gather);
          store(g, acc);
        } else {
          rest |= bit;
        }
        e0 = f0;
        e1 = f1;
        f0 = g0;
        f1 = g1;
        b0 = nb0;
        cnt = ncnt;
      }
    }
    if (rest == 0) continue;
    auto take = [&]() {  // the next of them, or -1
      if (rest == 0) return (int64_t)-1;
      const int64_t g = base + (int64_t)(__ffsll((unsigned long long)rest) - 1) * step;
      rest &= rest - 1;
      return g;
    };
    // entries of a row per pass: passes as even as whole batches of gathers allow
    auto pass_len = [&](int m) {
#pragma unroll
      for (int o = G; o < 64; o *= 2) m = max(m, __shfl_xor(m, o));
      m = __builtin_amdgcn_readfirstlane(m);  // the longest row, above kRowCap
      const int passes = (m - 1) / kRowPass + 1;
      return min(kRowPass, ((m - 1) / passes + 4) & ~3);
    };
    // (one entry more between the rows' parts: they start on different banks)
    static_assert(kRowPass < kRowCap && kRowPass % 4 == 0, "the rows' parts fit");
    Entry<TW>* x = E + r * (kRowPass + 1);
    int64_t g = take(), h = take();  // this group and the next
    load_rp(g, e0, e1);
    load_rp(h < 0 ? g : h, f0, f1);
    int32_t pc[NQ];
    TV pv[NQ];
    const int32_t* cp = ci + e0;
    const TV* vp = val + e0;
    int left = e1 - e0, len = pass_len(left);  // of the row (below 0 past its end), of the pass
    fetch(pc, pv, cp, vp, l, by_row, min(left, len));
    VT acc = zero();
    for (;;) {
      const int m = min(left, len);
      stage(pc, pv, x, l, by_row, m);
      const bool more = __ballot(left > len) != 0;
      if (more) {
        left -= len;
        cp += len;
        vp += len;
      } else {
        left = f1 - f0;
        len = pass_len(left);
        cp = ci + f0;
        vp = val + f0;
      }
      if (more || h >= 0) fetch(pc, pv, cp, vp, l, by_row, min(left, len));
      lds_ready();
      add_entries<CPL>(x, m, acc, gather);
      if (!more) {
        store(g, acc);
        if (h < 0) break;
        acc = zero();
        g = h;
        h = take();
        load_rp(h < 0 ? g : h, f0, f1);
      }
    }
  }
}

// The two kernels above, G lanes to a row, by the mean number of entries per row
// (the matrices measured have 4e7 entries or 1e6 rows, lengths +- 11 %; us, with
// 16 KB of LDS k_spmm_block : k_spmm_rows).
//   * Rows that mostly fit kRowCap: k_spmm_rows, whose loads overlap its gathers
//     (fp64, 16 columns: 27 entries 233 : 229, 41 343 : 315, 45 343 : 330, 47
//     341 : 404; 8 columns: 16 entries 127 : 115, 41 297 : 244; fp32, 16
//     columns: 16 entries 84 : 100, 20 137 : 126, 41 269 : 233), but not with 16
//     lanes per row (fp64, 32 columns, 41 entries: 547 : 605) or 8 in fp32 (292 :
//     308), where four to eight rows per wave are too little work per step.
//   * Short rows, and rows that do not fit: k_spmm_block, by more rows in flight
//     (fp64, 16 columns: 3 entries 74 : 87, 50 340 : 428, 64 327 : 412; rows of
//     random length, mean 41: 543 : 640).
//   * Rows so long that a block's take many passes, each as long as its longest
//     part of a row: k_spmm_rows (fp64, 16 columns: 128 entries 367 : 390, 144
//     437 : 400; 8: 160 398 : 430, 192 486 : 430; 32: 160 549 : 570, 192 577 :
//     562; fp32, 16: 224 390 : 408, 256 432 : 409; 32: 256 366 : 384, 512 659 :
//     380).
//   * Products that the waves on the chip take in one step (nothing to balance,
//     all latency; n = 20000, 16 fp64 columns, 41 entries 11 : 9, 96 30 : 20),
//     and of longer rows also those that the cache holds (n = 80000, 96 entries
//     82 : 60; 32 columns, n = 1e5, 100 entries 107 : 111, 140 160 : 151; 32 fp32
//     columns, n = 6e4, 150 62 : 62, 170 84 : 69), which do not wait for HBM.

// LDS of a workgroup of k_spmm_block, of `blocks`, whose rows have `entries`
// entries of `size` bytes on average: 20 KB, with which eight workgroups just
// share a CU; 26 where that saves a pass and the grid is many rounds or one; 16
// where the passes are as many and it is one, or they are nearly full, or the
// grid is two rounds (fp64, n = 3e5 or 4e5, 16 / 20 / 26 KB: 24 columns, 70
// entries per row 368 / 311 / 328 us, 80 403 / 344 / 354, 90 338 / 341 / 304, 110
// 416 / 381 / 392; 16 columns, 64 185 / 196 / 201, 80 256 / 212 / 244, 100 268 /
// 240 / 222; n = 6e4, 50 27 / 29; 32 fp32 columns, n = 1e6, 3 72 / 78).
static unsigned block_lds(double entries, int size, int64_t blocks) {
  auto passes = [&](int kb) { return std::ceil(entries * size / (kb * 1024.0)); };
  const bool few = blocks <= 12 * 256;
  if ((!few || blocks <= 6 * 256) && passes(26) < passes(20)) return 26 * 1024;
  if (passes(16) == passes(20) && (few || passes(16) <= 1 || entries * size > 0.9 * 16384 * passes(16)))
    return 16 * 1024;
  return 20 * 1024;
}

template <typename TV, typename TW, int G>
static hipError_t spmm_stream_launch(const int32_t* rp, const int32_t* ci, const TV* val, const TW* W,
                                     int64_t ldw, TW* Y, int64_t ldy, int ncols, int64_t n,
                                     int64_t nnz, int64_t between, hipStream_t s) {
  constexpr int CPL = 16 / (int)sizeof(TW);
  constexpr int NR = 64 / G, RPB = 256 / G;
  constexpr bool F64 = sizeof(TW) == 8;
  const int64_t groups = (n + NR - 1) / NR;
  const double mean = (double)nnz / (double)n;
  const bool big = (uint64_t)n * (uint64_t)ldw * sizeof(TW) >= (1ull << 32);
  // A matrix that the memory-side cache still holds at the next product is read
  // through the caches; a larger one, or one with too much between two products,
  // would only evict W and itself, and is read with the non-temporal hint.  What
  // passes: the matrix, W and Y, or what the caller names.  (One product after
  // another, 16 columns, with : without the hint: n = 1e6, 8 fp64 entries per row,
  // 356 MB 102 : 111 us; fp32 the same 192 MB 68 : 51, 16 entries 260 MB 114 : 84,
  // 20 entries 292 MB 136 : 138; n = 2e5, 80 fp64 entries, 24 columns 269 MB 169 :
  // 203, 32 columns 294 MB 212 : 205.  Whole fp64 solves of 41 entries per row, 12
  // columns: n = 1e5, 164 MB with the bases 9.50 : 9.40 ms; 2e5, 328 MB 14.04 :
  // 14.52; 3e5 29.6 : 30.0.)
  const int64_t product = 2 * n * ncols * (int64_t)sizeof(TW);
  const bool nt = big || nnz * (int64_t)(sizeof(TV) + 4) + std::max(product, between) > kCacheBytes;
  // (mean entries per row)
  constexpr int lo = G == 4 ? (F64 ? 14 : 18) : (F64 && G == 8) ? 30 : INT_MAX;
  constexpr int hi = F64 ? (G == 8 ? 138 : 176) : (G == 4 ? 240 : 288);
  // (6000 to 9400 groups are one to two rounds of k_spmm_block's workgroups, the
  // last one uneven: 23 fp32 columns, n = 7e4, 41 entries per row 27 : 29 us)
  const bool waves = (groups <= 16 * 256 && mean >= 14) || (mean >= lo && mean <= 45.5) ||
                     (G == 8 && groups > 6000 && groups <= 9400 && mean > 20 && mean <= 45.5) ||
                     (!nt && ((F64 && mean > (G <= 8 ? 56 : groups <= 9400 ? 75 : 105)) || (G == 8 && mean > 155) ||
                              (groups <= 9400 && mean > 160))) ||
                     mean > hi;
  auto launch = [&](auto kernel, int64_t nb, int64_t units, unsigned lds, auto... more) {
    const unsigned grid = (unsigned)((nb + 7) / 8 * 8);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds, s, rp, ci, val, W, ldw, Y, ldy, ncols, n,
                       (int)((units + 7) / 8), more...);
    return hipGetLastError();
  };
  if (waves) {
    // a persistent grid, a multiple of the 8 XCDs: four workgroups per CU, three
    // where a wave takes 16 rows (their registers and LDS)
    const int64_t nb = std::min<int64_t>((groups + 3) / 4, 256 * kRowsWaves(G));
    if (big) return launch(k_spmm_rows<TV, TW, G, CPL, true, true>, nb, groups, 0);
    if (nt) return launch(k_spmm_rows<TV, TW, G, CPL, false, true>, nb, groups, 0);
    return launch(k_spmm_rows<TV, TW, G, CPL, false, false>, nb, groups, 0);
  }
  const int64_t nb = (n + RPB - 1) / RPB;
  const unsigned lds = block_lds(mean * RPB, sizeof(Entry<TW>), nb), cap = lds / (unsigned)sizeof(Entry<TW>);
  if (big) return launch(k_spmm_block<TV, TW, G, CPL, true, true>, nb, nb, lds, cap);
  if (nt) return launch(k_spmm_block<TV, TW, G, CPL, false, true>, nb, nb, lds, cap);
  return launch(k_spmm_block<TV, TW, G, CPL, false, false>, nb, nb, lds, cap);
}

// ---- banded matrices: W staged in LDS, slab by slab ----
// A workgroup of kSlabThreads takes kSlabBlockRows consecutive rows (4 lanes
// per row, 4 of the 16 columns per lane, kSlabUnits rows per thread).  The W
// rows that its entries reference lie in the block's column window
// [win.x, win.y] (computed once per operator); it walks that window in slabs
// of kSlabLds bytes (1024 fp64 or 2048 fp32 W rows of 16 columns), staging
// each slab in LDS once, and every row consumes the entries whose column
// falls in the slab (its columns are sorted, so they are the next ones of the
// row).  The W gathers then come from LDS, but each (col, val) load now
// reads 16 rows' entries at once, slab after slab: on the n = 1e6 banded
// matrix (band +-5000, 16 fp64 columns) this path takes 1.4 ms against the
// gather kernel's 0.38 ms (2.6 ms when every row's next entry was loaded
// together per round), so it is not the default (LOBPCG_OPT_SPMM_SLAB).
template <typename TV, typename TW>
__global__ __launch_bounds__(kSlabThreads) void k_spmm_slab(const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ ci,
                                                            const TV* __restrict__ val,
                                                            const TW* __restrict__ W, int64_t ldw,
                                                            TW* __restrict__ Y, int64_t ldy,
                                                            int ncols, int64_t n,
                                                            const int2* __restrict__ win,
                                                            int per_xcd) {
  // W rows in LDS at a stride of 17 elements: the 16 rows a wave reads at
  // once then start on different banks (at 16 they shared two bank groups)
  constexpr int LS = 17;
  constexpr int SW = kSlabLds / (LS * (int)sizeof(TW));  // W rows per slab
  constexpr int U = kSlabUnits;
  constexpr int RG = kSlabThreads / 4;  // rows taken at once
  extern __shared__ char slab_smem[];
  TW* Ws = reinterpret_cast<TW*>(slab_smem);
  const int b = blockIdx.x;
  const int lb = (b & 7) * per_xcd + (b >> 3);  // XCD b % 8 walks a contiguous range
  const int64_t r0 = (int64_t)lb * kSlabBlockRows;
  if (r0 >= n) return;  // whole block
  const int lane = threadIdx.x & 3, rg = threadIdx.x >> 2;
  int p[U], e[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = r0 + rg + (int64_t)RG * u;
    p[u] = (i < n) ? rp[i] : 0;
    e[u] = (i < n) ? rp[i + 1] : 0;
  }
  TW acc[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[u][q] = TW(0);
  const int2 w = win[lb];
  if (w.y >= w.x) {
    const int s_lo = w.x / SW, s_hi = w.y / SW;
    for (int s = s_lo; s <= s_hi; ++s) {
      const int64_t c0 = (int64_t)s * SW;
      __syncthreads();  // the previous slab is consumed
      for (int q = threadIdx.x; q < SW * 16; q += kSlabThreads) {
        const int rr = q >> 4, cc = q & 15;
        const int64_t wr = c0 + rr;
        Ws[rr * LS + cc] = (wr < n && cc < ncols) ? W[wr * ldw + cc] : TW(0);
      }
      __syncthreads();
      const int64_t cend = c0 + SW;
      // each row takes its next entries while their columns lie in this slab
#pragma unroll
      for (int u = 0; u < U; ++u) {
        while (p[u] < e[u]) {
          const int col = ci[p[u]];
          if (col >= cend) break;
          const TW v = (TW)val[p[u]];
          const TW* wr = Ws + (col - c0) * LS + 4 * lane;
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[u][q] += v * wr[q];
          ++p[u];
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = r0 + rg + (int64_t)RG * u;
    if (i < n) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 4 * lane + q;
        if (c < ncols) Y[i * ldy + c] = acc[u][q];
      }
    }
  }
}

template <typename TV, typename TW>
static hipError_t spmm_slab_launch(const int32_t* rp, const int32_t* ci, const TV* val,
                                   const TW* W, int64_t ldw, TW* Y, int64_t ldy, int ncols,
                                   int64_t n, const int2* win, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_spmm_slab<TV, TW>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kSlabLds);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const int64_t nb = (n + kSlabBlockRows - 1) / kSlabBlockRows;
  const int64_t nbp = (nb + 7) / 8 * 8;
  hipLaunchKernelGGL((k_spmm_slab<TV, TW>), dim3((unsigned)nbp), dim3(kSlabThreads), kSlabLds, s,
                     rp, ci, val, W, ldw, Y, ldy, ncols, n, win, (int)(nbp / 8));
  return hipGetLastError();
}

// Column window of each kSlabBlockRows-row block: win[b] = (smallest first
// column, largest last column) over its rows, (INT_MAX, -1) for a block of
// empty rows; *unsorted = 1 if some row's columns decrease.
__global__ __launch_bounds__(256) void k_csr_windows(const int32_t* __restrict__ rp,
                                                     const int32_t* __restrict__ ci, int64_t n,
                                                     int2* __restrict__ win,
                                                     int* __restrict__ unsorted) {
  __shared__ int slo[256], shi[256];
  const int64_t r0 = (int64_t)blockIdx.x * kSlabBlockRows;
  const int64_t r1 = min(n, r0 + kSlabBlockRows);
  int lo = INT_MAX, hi = -1;
  bool bad = false;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += 256) {
    const int a = rp[i], z = rp[i + 1];
    if (z > a) {
      lo = min(lo, ci[a]);
      hi = max(hi, ci[z - 1]);
      for (int q = a + 1; q < z; ++q) bad |= ci[q] < ci[q - 1];
    }
  }
  if (bad) *unsorted = 1;
  slo[threadIdx.x] = lo;
  shi[threadIdx.x] = hi;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) {
      slo[threadIdx.x] = min(slo[threadIdx.x], slo[threadIdx.x + w]);
      shi[threadIdx.x] = max(shi[threadIdx.x], shi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) win[blockIdx.x] = make_int2(slo[0], shi[0]);
}

template <typename TV, typename TW>
static hipError_t spmm_any(const int32_t* rp, const int32_t* ci, const TV* val, const TW* W,
                           int64_t ldw, TW* Y, int64_t ldy, int ncols, int64_t n, int64_t nnz,
                           int64_t between, const int2* win, hipStream_t s) {
  if (n < 1 || ncols < 1) return hipErrorInvalidValue;
  if (win != nullptr) {
    for (int c0 = 0; c0 < ncols; c0 += 16) {
      hipError_t e = spmm_slab_launch<TV, TW>(rp, ci, val, W + c0, ldw, Y + c0, ldy,
                                              std::min(16, ncols - c0), n, win, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  constexpr int CPL = 16 / (int)sizeof(TW);
  // the 16-byte kernels are used from 5 (fp64) / 9 (fp32) columns, below which
  // the one-column-per-lane kernel is as fast, up to 16 lanes per row.  Five to
  // eight fp64 columns that are not aligned to 16 bytes stay with the latter,
  // which adds the entries of a row in two sums, and where these are the end of
  // 33 to 40 they go to the former, which add in order: a solve that has not
  // converged amplifies rounding, so each product keeps its order of addition.
  // Nine to sixteen misaligned fp32 columns of longer rows go to the latter too:
  // a gather of theirs by four lanes touches two lines as often as not, one by
  // sixteen lanes once (us, it : the others: 13 columns, n = 5e4, 41 entries per
  // row 17.5 : 19.1, 60 24 : 30, 80 30 : 38; n = 1e5, 80 55 : 63; n = 2e5 103 :
  // 110, but n = 3e5, 60 121 : 116, n = 25000, 80 17.7 : 16.9 and n = 1.4e5, 41 43 :
  // 41; 9 columns, n = 5e4, 60 22.6 : 26.6; 10, n = 37000, 60 17.8 : 16.4, 80 22.3 :
  // 23.5).
  const bool mis = (reinterpret_cast<uintptr_t>(W) % 16) != 0 || ldw % CPL != 0;
  const double mean = (double)nnz / (double)n;
  auto longer = [&](int nc) {
    if (n > 200000 || (n > 15000 && n < 30000)) return false;
    if (nc >= 13 && n > 44000 && n < 110000) return mean > 24;
    return mean > ((nc >= 13 || (n > 44000 && n <= 65536)) ? 45.5 : 70.0);
  };
  const bool odd = CPL == 2 && mis;
  const int wide_min = (CPL == 2) ? (odd ? 9 : 5) : 9;
  constexpr int slice = 16 * CPL;
  for (int c0 = 0; c0 < ncols; c0 += slice) {
    int nc = std::min(slice, ncols - c0), c = c0;
    const bool tail = odd && c0 > 0;
    if (tail && nc == 1) {  // with its neighbour, which takes the same value again
      nc = 2;
      c = c0 - 1;
    }
    const TW* Wc = W + c;
    TW* Yc = Y + c;
    hipError_t e;
    if (CPL == 4 && mis && nc > 8 && nc <= 16 && longer(nc)) {
      e = spmm_launch<TV, TW, 16>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, s);
    } else if (nc >= wide_min || tail) {
      const int lanes = (nc + CPL - 1) / CPL;
      if (lanes <= 4) e = spmm_stream_launch<TV, TW, 4>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, nnz, between, s);
      else if (lanes <= 8) e = spmm_stream_launch<TV, TW, 8>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, nnz, between, s);
      else e = spmm_stream_launch<TV, TW, 16>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, nnz, between, s);
    } else if (nc <= 1) e = spmm_launch<TV, TW, 1>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, s);
    else if (nc <= 2) e = spmm_launch<TV, TW, 2>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, s);
    else if (nc <= 4) e = spmm_launch<TV, TW, 4>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, s);
    else e = spmm_launch<TV, TW, 8>(rp, ci, val, Wc, ldw, Yc, ldy, nc, n, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t spmm_csr_f64(const int32_t* rp, const int32_t* ci, const double* val, const double* W,
                        int64_t ldw, double* Y, int64_t ldy, int ncols, int64_t n, int64_t nnz,
                        int64_t between, const int2* win, hipStream_t s) {
  return spmm_any<double, double>(rp, ci, val, W, ldw, Y, ldy, ncols, n, nnz, between, win, s);
}
hipError_t spmm_csr_f32(const int32_t* rp, const int32_t* ci, const float* val, const float* W,
                        int64_t ldw, float* Y, int64_t ldy, int ncols, int64_t n, int64_t nnz,
                        int64_t between, const int2* win, hipStream_t s) {
  return spmm_any<float, float>(rp, ci, val, W, ldw, Y, ldy, ncols, n, nnz, between, win, s);
}
hipError_t csr_windows(const int32_t* rp, const int32_t* ci, int64_t n, int2* win, int* unsorted,
                       hipStream_t s) {
  const int64_t nb = (n + kSlabBlockRows - 1) / kSlabBlockRows;
  if (nb < 1) return hipSuccess;
  hipLaunchKernelGGL(k_csr_windows, dim3((unsigned)nb), dim3(256), 0, s, rp, ci, n, win, unsorted);
  return hipGetLastError();
}

}  // namespace lobpcg
