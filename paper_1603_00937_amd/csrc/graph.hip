// Spectral bounds, the SP2 start map X0, and the data-dependency graphs (Eq. 2, Eq. 8,
// obs. viii).  Every floating-point result that decides an integer (a graph edge) is
// evaluated in a canonical order with separately rounded operations, so the graph is the
// same bit for bit as a sequential CPU evaluation: Gershgorin row sums in ascending column
// order, x0 = (e_max*delta_ij - h_ij)/(e_max - e_min), and (X0^2)_ij accumulated over k in
// ascending order.  The library is compiled with floating-point contraction disabled.
#include "internal.h"
#include "lds_hash.h"
#include "lds_scan.h"

#include <cstdlib>
#include <map>
#include <string>
#include <mutex>

#pragma clang fp contract(off)

namespace gbi {
namespace {

constexpr int kT = 256;

__device__ __forceinline__ double x0_entry(double h, bool diag, double emax, double denom) {
  const double num = diag ? (emax - h) : (0.0 - h);
  return num / denom;
}

// Gershgorin row ends lo_i = h_ii - R_i, hi_i = h_ii + R_i, with R_i = sum_{j != i} |h_ij| summed
// in slot (ascending column) order up to the first padding entry.  The order makes a row's sum a
// serial chain, so what can be had is coalesced loads and many rows at once: a wave takes
// kDiscRows rows, 64 slots of each at a time through LDS (its next slots are in registers
// meanwhile), and one lane per row adds them up.  The row ends are reduced per workgroup (row
// groups grid-strided) into (min lo, max hi, rows with an end that is not finite) partials, then
// by one workgroup: min and max are exact, so the order does not matter.  A NaN or Inf anywhere in
// a row makes its ends so; fmin / fmax alone would skip a NaN.  Padding at the end of rows is read
// 64 slots past the longest row of the group, no further (N = 4096, 247 of 2247 slots used: 0.17 ->
// 0.05 ms).
// One thread per row straight from memory took 185 us at N = 18000 (255 slots) and 45 us at 256;
// this takes 30 and 17 (128 us at N = 100000 x 335, 3.1 TB/s).
constexpr int kDiscRows = 16;
constexpr int kDiscGroup = kDiscRows * (kT / 64);  // rows per workgroup and round

// The allocation-free bounds keep partials and result in `scratch`, a fixed device array: each
// workgroup writes its own three entries before the final pass reads them, so nothing has to
// start at zero.
constexpr int kNoallocBlocks = 1024;
static __device__ __align__(256) double scratch[3 * kNoallocBlocks + 3];

__device__ __forceinline__ void reduce3(double& a, double& b, double& c, double* sa, double* sb,
                                        double* sc) {
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  sc[threadIdx.x] = c;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      sa[threadIdx.x] = fmin(sa[threadIdx.x], sa[threadIdx.x + h]);
      sb[threadIdx.x] = fmax(sb[threadIdx.x], sb[threadIdx.x + h]);
      sc[threadIdx.x] += sc[threadIdx.x + h];
    }
    __syncthreads();
  }
  a = sa[0];
  b = sb[0];
  c = sc[0];
}

__global__ __launch_bounds__(kT) void k_disc_partials(const int32_t* __restrict__ col,
                                                      const double* __restrict__ val, int n, int w,
                                                      double* __restrict__ part) {
  __shared__ double sv[kT / 64][kDiscRows][65];
  __shared__ int32_t sc[kT / 64][kDiscRows][65];
  __shared__ double sa[kT], sb[kT], sd[kT];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double a = INFINITY, b = -INFINITY, bad = 0.0;
  for (int64_t g = blockIdx.x; g * kDiscGroup < n; g += gridDim.x) {
    const int64_t r0 = g * kDiscGroup + wave * kDiscRows;
    const int64_t i = r0 + lane;
    double r = 0.0, d = 0.0;
    bool open = lane < kDiscRows && i < n;
    int32_t c[kDiscRows];
    double v[kDiscRows];
    auto load = [&](int t0) {
#pragma unroll
      for (int q = 0; q < kDiscRows; ++q) {
        const bool in = r0 + q < n && t0 + lane < w;
        const int64_t e = in ? (r0 + q) * w + t0 + lane : 0;
        c[q] = in ? col[e] : -1;
        v[q] = in ? val[e] : 0.0;
      }
    };
    load(0);
    for (int t0 = 0; t0 < w; t0 += 64) {
      // every row of the group has ended: what is left is padding
      if (!__syncthreads_or(t0 == 0 || open)) break;
#pragma unroll
      for (int q = 0; q < kDiscRows; ++q) {
        sc[wave][q][lane] = c[q];
        sv[wave][q][lane] = v[q];
      }
      __syncthreads();
      if (t0 + 64 < w) load(t0 + 64);
      if (lane < kDiscRows) {
#pragma unroll
        for (int t8 = 0; t8 < 64; t8 += 8) {
          int32_t j[8];
          double x[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            j[q] = sc[wave][lane][t8 + q];
            x[q] = sv[wave][lane][t8 + q];
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) {  // adding 0 changes no bit of a sum of magnitudes
            open = open && j[q] >= 0;
            d = open && j[q] == i ? x[q] : d;
            r = r + (open && j[q] != i ? fabs(x[q]) : 0.0);
          }
        }
      }
    }
    if (lane < kDiscRows && i < n) {
      const double lo = d - r, hi = d + r;
      if (!isfinite(lo) || !isfinite(hi)) bad += 1.0;
      a = fmin(a, lo);
      b = fmax(b, hi);
    }
  }
  reduce3(a, b, bad, sa, sb, sd);
  if (threadIdx.x == 0) {
    part[3 * blockIdx.x] = a;
    part[3 * blockIdx.x + 1] = b;
    part[3 * blockIdx.x + 2] = bad;
  }
}

__global__ __launch_bounds__(kT) void k_disc_final(const double* __restrict__ part, int nb,
                                                   double* __restrict__ out) {
  __shared__ double sa[kT], sb[kT], sc[kT];
  double a = INFINITY, b = -INFINITY, bad = 0.0;
  for (int q = threadIdx.x; q < nb; q += kT) {
    a = fmin(a, part[3 * q]);
    b = fmax(b, part[3 * q + 1]);
    bad += part[3 * q + 2];
  }
  reduce3(a, b, bad, sa, sb, sc);
  if (threadIdx.x == 0) {
    out[0] = a;
    out[1] = b;
    out[2] = bad;
  }
}

__global__ void k_x0(const int32_t* __restrict__ col, const double* __restrict__ val, int n, int w,
                     double emax, double denom, double* __restrict__ x0) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (int64_t)n * w) return;
  const int i = (int)(p / w);
  const int32_t j = col[p];
  x0[p] = j < 0 ? 0.0 : x0_entry(val[p], j == i, emax, denom);
}

// ---- X2 graph, one workgroup per row i --------------------------------------------------
// The edge (i, j) is decided by |(X0^2)_ij| >= tau, the entry summed over k in row i in
// ascending order (row i's slots in order), every product and sum rounded separately.  The
// kernels accumulate the entries with LDS atomic adds instead, in whatever order the adds
// land, with no barrier between the rows k, and keep that order's result only where it cannot
// change the decision: two summation orders of the same m rounded products p_k differ by at
// most 2 gamma_{m-1} sum |p_k| (gamma_m = m u / (1 - m u), u = 2^-53; the standard bound on
// recursive summation), and sum_k |x0_ik x0_kj| <= b_i = sum_k |x0_ik| max_l |x0_kl|.  A
// candidate with | |acc| - tau | within twice that of tau (at most a few per graph, usually
// none) is summed again in ascending order by one wave, so the graph is the one of the
// ascending sums bit for bit.
//   1. mark every j in row k for every k in row i (two-hop candidates) and i itself;
//   2. rank = number of candidates below j (per-word popcount prefix);
//   3. acc[rank(j)] += x0_ik * x0_kj over every (k, j), LDS atomic adds;
//   4. keep j if j == i or |acc| >= tau (re-summed in ascending order near tau): the count,
//      and the sorted columns into the row's slot of a staging array (cap entries per row;
//      k_x2_compact then packs them into the CSR), so the product is computed once.
// LDS: candidate bitmap over all n vertices, per-word rank base, accumulators of the
// candidates (indexed by rank), and row i's columns / x0 values.
struct X2Lds {
  uint32_t* bits;
  int32_t* pre;
  double* acc;
  int32_t* ci;
  double* xi;
};

constexpr int kX2Q = 4;  // ELL width limit: kX2Q * kT (the float index split below needs < 2048)
constexpr int kX2B = 8;  // (k, j) pairs whose loads a thread has in flight at once

// the (slot t of row i, slot u of row k) pair number p = t w + u, split without an integer
// division: (p + 0.5) / w is at least 0.5 / w away from an integer and p < w^2 < 2^22, so the
// float quotient truncates to t (the correction below is a guard)
__device__ __forceinline__ void x2_pair(int p, int w, float inv_w, int& t, int& u) {
  t = (int)(((float)p + 0.5f) * inv_w);
  u = p - t * w;
  if (u < 0) {
    --t;
    u += w;
  } else if (u >= w) {
    ++t;
    u -= w;
  }
}

// the rows k of row i are its slots before the first padding entry
__device__ __forceinline__ int x2_row_width(const int32_t* ci, int w, int n, int32_t* red) {
  if (threadIdx.x == 0) red[0] = w;
  __syncthreads();
  for (int t = threadIdx.x; t < w; t += kT)
    if ((unsigned)ci[t] >= (unsigned)n) atomicMin(&red[0], t);
  __syncthreads();
  const int kw = red[0];
  __syncthreads();  // red is reused
  return kw;
}

// step 1 and step 3 over the kw * w pairs: mark(j), or add(j, x0_ik * x0_kj)
template <bool ADD, class F>
__device__ __forceinline__ void x2_pairs(const int32_t* __restrict__ hcol,
                                         const double* __restrict__ x0, const int32_t* ci,
                                         const double* xi, int kw, int w, float inv_w, int n,
                                         F&& f) {
  const int npair = kw * w;
  for (int p0 = threadIdx.x; p0 < npair; p0 += kX2B * kT) {
    int32_t jj[kX2B];
    double xk[kX2B], xx[kX2B];  // x0_ik, x0_kj
#pragma unroll
    for (int q = 0; q < kX2B; ++q) {  // every load of the batch first
      const int p = p0 + q * kT;
      jj[q] = -1;
      xk[q] = xx[q] = 0.0;
      if (p < npair) {
        int t, u;
        x2_pair(p, w, inv_w, t, u);
        const int64_t e = (int64_t)ci[t] * w + u;
        jj[q] = hcol[e];
        if (ADD) {
          xx[q] = x0[e];
          xk[q] = xi[t];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kX2B; ++q)
      if ((unsigned)jj[q] < (unsigned)n) f(jj[q], ADD ? xk[q] * xx[q] : 0.0);
  }
}

// the half-width of the band around tau in which the order of the sum may decide (see above):
// twice the bound, b_i rounded, a term for underflow
__device__ __forceinline__ double x2_margin(int kw, double b, double tau) {
  return (4.0 * kw + 8.0) * 0x1p-53 * b + 4.0 * 0x1p-53 * tau + 1e-300;
}

// (X0^2)_ij summed in ascending order of row i's slots, every product and sum rounded
// separately, by a whole wave: lane l looks j up in the rows k of slots l, l + 64, ... (a scan
// of the row, which assumes nothing of its order) and the products are added one slot after
// the other.
__device__ double x2_sum_ascending(const int32_t* __restrict__ hcol,
                                   const double* __restrict__ x0, const int32_t* ci,
                                   const double* xi, int kw, int w, int32_t j) {
  const int lane = threadIdx.x & 63;
  double acc = 0.0;
  for (int t0 = 0; t0 < kw; t0 += 64) {
    const int t = t0 + lane;
    double prod = 0.0;
    int found = 0;
    if (t < kw) {
      const int64_t base = (int64_t)ci[t] * w;
      for (int u = 0; u < w; ++u)
        if (hcol[base + u] == j) {
          found = 1;
          prod = xi[t] * x0[base + u];
          break;
        }
    }
    const int m = min(64, kw - t0);
    for (int l = 0; l < m; ++l)
      if (__shfl(found, l)) acc = acc + __shfl(prod, l);
  }
  return acc;
}

__global__ __launch_bounds__(kT) void k_x2_rows(const int32_t* __restrict__ hcol,
                                                const double* __restrict__ x0,
                                                const double* __restrict__ rbound, int n, int w,
                                                float inv_w, double tau, int all_ascending,
                                                int cap, int32_t* __restrict__ cnt,
                                                int32_t* __restrict__ rows,
                                                int32_t* __restrict__ overflow) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t nband;
  const int i = blockIdx.x;
  const int nw = (n + 31) >> 5;
  X2Lds L;
  L.acc = reinterpret_cast<double*>(smem);
  L.xi = L.acc + cap;
  L.bits = reinterpret_cast<uint32_t*>(L.xi + w);
  L.pre = reinterpret_cast<int32_t*>(L.bits + nw);
  L.ci = L.pre + nw + 1;
  int32_t* red = L.ci + w;  // kT ints

  for (int t = threadIdx.x; t < w; t += kT) {
    L.ci[t] = hcol[(int64_t)i * w + t];
    L.xi[t] = x0[(int64_t)i * w + t];
  }
  for (int q = threadIdx.x; q < nw; q += kT) L.bits[q] = 0u;
  if (threadIdx.x == 0) nband = 0;
  const int kw = x2_row_width(L.ci, w, n, red);
  // 1. two-hop candidates
  x2_pairs<false>(hcol, x0, L.ci, L.xi, kw, w, inv_w, n, [&](int32_t j, double) {
    atomicOr(&L.bits[j >> 5], 1u << (j & 31));
  });
  if (threadIdx.x == 0) atomicOr(&L.bits[i >> 5], 1u << (i & 31));
  __syncthreads();
  // 2. ranks
  for (int q = threadIdx.x; q < nw; q += kT) L.pre[q] = __popc(L.bits[q]);
  __syncthreads();
  const int32_t ncand = lds_exclusive_scan<kT>(L.pre, nw, red);
  if (ncand > cap) {
    if (threadIdx.x == 0) {
      atomicMax(overflow, ncand);
      cnt[i] = 0;
    }
    return;
  }
  for (int r = threadIdx.x; r < ncand; r += kT) L.acc[r] = 0.0;
  __syncthreads();
  // 3. accumulation, adds in any order
  x2_pairs<true>(hcol, x0, L.ci, L.xi, kw, w, inv_w, n, [&](int32_t j, double prod) {
    const uint32_t word = L.bits[j >> 5];
    const int r = L.pre[j >> 5] + __popc(word & ((1u << (j & 31)) - 1u));
    atomicAdd(&L.acc[r], prod);
  });
  __syncthreads();
  // 4. decisions: bits[q] becomes the word's kept set, pre[q] (no longer needed for ranks)
  //    its candidates near tau, then its kept count
  const double margin = x2_margin(kw, rbound[i], tau);
  for (int q = threadIdx.x; q < nw; q += kT) {
    uint32_t word = L.bits[q], keep = 0u, band = 0u;
    int r = L.pre[q];
    while (word) {
      const int b = __ffs(word) - 1;
      const int j = (q << 5) + b;
      const double a = fabs(L.acc[r]);
      if (j == i) keep |= 1u << b;
      else if (all_ascending || fabs(a - tau) <= margin) band |= 1u << b;
      else if (a >= tau) keep |= 1u << b;
      ++r;
      word &= word - 1u;
    }
    L.bits[q] = keep;
    L.pre[q] = (int32_t)band;
    if (band) atomicAdd(&nband, __popc(band));
  }
  __syncthreads();
  if (nband > 0) {
    // ascending sums of the candidates near tau, one wave per word
    for (int q = threadIdx.x >> 6; q < nw; q += kT / 64) {
      uint32_t band = (uint32_t)L.pre[q];
      while (band) {
        const int b = __ffs(band) - 1;
        const double a = fabs(x2_sum_ascending(hcol, x0, L.ci, L.xi, kw, w, (q << 5) + b));
        if ((threadIdx.x & 63) == 0 && a >= tau) atomicOr(&L.bits[q], 1u << b);
        band &= band - 1u;
      }
    }
    __syncthreads();
  }
  for (int q = threadIdx.x; q < nw; q += kT) L.pre[q] = __popc(L.bits[q]);
  __syncthreads();
  const int32_t kept = lds_exclusive_scan<kT>(L.pre, nw, red);
  if (threadIdx.x == 0) cnt[i] = kept;
  int32_t* dst = rows + (int64_t)i * cap;  // kept <= ncand <= cap
  for (int q = threadIdx.x; q < nw; q += kT) {
    uint32_t word = L.bits[q];
    int32_t pos = L.pre[q];
    while (word) {
      const int b = __ffs(word) - 1;
      dst[pos++] = (q << 5) + b;
      word &= word - 1u;
    }
  }
}

// max_l |x0_kl| of every row k, and the slots up to its last entry (one wave per row)
__global__ __launch_bounds__(kT) void k_row_absmax(const int32_t* __restrict__ col,
                                                   const double* __restrict__ x0, int n, int w,
                                                   double* __restrict__ out,
                                                   int32_t* __restrict__ rlen) {
  const int row = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  double m = 0.0;
  int len = 0;
  for (int u = lane; u < w; u += 64) {
    m = fmax(m, fabs(x0[(int64_t)row * w + u]));
    if ((unsigned)col[(int64_t)row * w + u] < (unsigned)n) len = u + 1;
  }
  for (int o = 32; o > 0; o >>= 1) {
    m = fmax(m, __shfl_xor(m, o));
    len = max(len, __shfl_xor(len, o));
  }
  if (lane == 0) {
    out[row] = m;
    rlen[row] = len;
  }
}

// b_i = sum over the slots of row i of |x0_ik| max_l |x0_kl|, which bounds sum_k |x0_ik x0_kj|
// for every j (one wave per row)
__global__ __launch_bounds__(kT) void k_x2_bound(const int32_t* __restrict__ col,
                                                 const double* __restrict__ x0,
                                                 const double* __restrict__ amax, int n, int w,
                                                 double* __restrict__ out) {
  const int row = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  double b = 0.0;
  for (int u = lane; u < w; u += 64) {
    const int64_t e = (int64_t)row * w + u;
    const int32_t k = col[e];
    if ((unsigned)k < (unsigned)n) b += fabs(x0[e]) * amax[k];
  }
  for (int o = 32; o > 0; o >>= 1) b += __shfl_xor(b, o);
  if (lane == 0) out[row] = b;
}

// The same rows for any n: the two-hop candidates of row i go into an LDS hash set instead of
// an n-bit bitmap and are sorted to fix their ranks; accumulation and decisions are those of
// k_x2_rows, so the graph is the same bit for bit.  LDS: acc [cap], x0 of row i [w], keys and
// their ranks [2^log2h each], the sorted candidates [2^log2u >= cap], columns of row i [w],
// scratch [kT].  Inserts stop once more than cap candidates were counted (at most kT more
// land, and 2^log2h >= cap + kT + 1 keeps the set from filling); such a row reports its count
// through `overflow`.
__global__ __launch_bounds__(kT) void k_x2_rows_hash(const int32_t* __restrict__ hcol,
                                                     const double* __restrict__ x0,
                                                     const double* __restrict__ rbound, int n,
                                                     int w, float inv_w, double tau,
                                                     int all_ascending, int cap, int log2h,
                                                     int log2u, int32_t* __restrict__ cnt,
                                                     int32_t* __restrict__ rows,
                                                     int32_t* __restrict__ overflow) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t count, gathered, nband;
  const int i = blockIdx.x;
  const int H = 1 << log2h, P = 1 << log2u;
  double* acc = reinterpret_cast<double*>(smem);
  double* xi = acc + cap;
  int32_t* keys = reinterpret_cast<int32_t*>(xi + w);
  int32_t* rk = keys + H;
  int32_t* U = rk + H;
  int32_t* ci = U + P;
  int32_t* red = ci + w;
  for (int t = threadIdx.x; t < w; t += kT) {
    ci[t] = hcol[(int64_t)i * w + t];
    xi[t] = x0[(int64_t)i * w + t];
  }
  for (int q = threadIdx.x; q < H; q += kT) keys[q] = kHashEmpty;
  if (threadIdx.x == 0) {
    count = 0;
    gathered = 0;
    nband = 0;
  }
  const int kw = x2_row_width(ci, w, n, red);
  // 1. two-hop candidates (and i itself)
  if (threadIdx.x == 0 && hset_insert(keys, log2h, i)) atomicAdd(&count, 1);
  x2_pairs<false>(hcol, x0, ci, xi, kw, w, inv_w, n, [&](int32_t j, double) {
    if (*(volatile int32_t*)&count <= cap && hset_insert(keys, log2h, j)) atomicAdd(&count, 1);
  });
  __syncthreads();
  const int ncand = count;
  if (ncand > cap) {
    if (threadIdx.x == 0) {
      atomicMax(overflow, ncand);
      cnt[i] = 0;
    }
    return;
  }
  // 2. ranks: the candidates sorted ascending
  for (int q = threadIdx.x; q < H; q += kT) {
    const int32_t k = keys[q];
    if (k != kHashEmpty) U[atomicAdd(&gathered, 1)] = k;
  }
  __syncthreads();
  for (int r = ncand + threadIdx.x; r < P; r += kT) U[r] = INT32_MAX;
  bitonic_sort<kT>(U, P);
  for (int r = threadIdx.x; r < ncand; r += kT) {
    rk[hset_find(keys, log2h, U[r])] = r;
    acc[r] = 0.0;
  }
  __syncthreads();
  // 3. accumulation, adds in any order
  x2_pairs<true>(hcol, x0, ci, xi, kw, w, inv_w, n, [&](int32_t j, double prod) {
    atomicAdd(&acc[rk[hset_find(keys, log2h, j)]], prod);
  });
  __syncthreads();
  // 4. decisions (rk reused: 1 kept, 0 dropped, 2 near tau), ascending sums near tau, ordered
  //    compaction
  const double margin = x2_margin(kw, rbound[i], tau);
  for (int r = threadIdx.x; r < ncand; r += kT) {
    const double a = fabs(acc[r]);
    int f;
    if (U[r] == i) f = 1;
    else if (all_ascending || fabs(a - tau) <= margin) f = 2;
    else f = a >= tau ? 1 : 0;
    rk[r] = f;
    if (f == 2) atomicAdd(&nband, 1);
  }
  __syncthreads();
  if (nband > 0) {
    for (int r = threadIdx.x >> 6; r < ncand; r += kT / 64) {
      if (rk[r] != 2) continue;  // uniform over the wave
      const double a = fabs(x2_sum_ascending(hcol, x0, ci, xi, kw, w, U[r]));
      if ((threadIdx.x & 63) == 0) rk[r] = a >= tau ? 1 : 0;
    }
    __syncthreads();
  }
  for (int r = threadIdx.x; r < ncand; r += kT) acc[r] = rk[r];  // the flags, for the writes
  __syncthreads();
  const int32_t kept = lds_exclusive_scan<kT>(rk, ncand, red);
  if (threadIdx.x == 0) cnt[i] = kept;
  int32_t* dst = rows + (int64_t)i * cap;
  for (int r = threadIdx.x; r < ncand; r += kT)
    if (acc[r] != 0.0) dst[rk[r]] = U[r];
}

// The same rows in one pass over the pairs: the accumulators themselves sit in LDS pages of
// 2^shift consecutive vertices, given out as row i's pairs first touch them (dir: page number ->
// LDS slot).  Vertices close in space are close in number, so the ~1500 candidates of a row touch
// few pages (about 160 of 32 vertices), and neither a candidate set nor ranks are needed: the sums
// start at -0, which the first product that is not -0 itself changes for good, so an entry that
// still holds it was reached by no pair, or sums to 0 in any order, and tau > 0 drops it.  (Were it
// +0, a tau below the rounding of the sums would have every such entry, half of the pages', summed
// once more: 17 ms instead of 0.3 at N = 1024, tau = 1e-15.)  The other decisions, and the sums
// near tau, are those of k_x2_rows, so the graph is the same bit for bit.  One wave takes a row k
// at a time, 64 slots per step up to the row's last entry.  A row that needs more than pcap pages
// or keeps more than cap entries reports it through `overflow` (pages, kept) and the launch is
// repeated with room or left to the kernels below; workgroups that start after a report of more
// than `most` pages, which ends the attempt for good, return at once (vertices numbered at random,
// N = 18000: 4.4 ms spent on two attempts before the two passes' 2.1, now 0.1).
// The two-pass kernels visit every pair twice with an LDS atomic and two LDS look-ups; here a
// pair costs one look-up and one ds_add_f64, and LDS no longer grows with n.  Bound by LDS and the
// vector work of a pair at two workgroups per CU (the pages take ~50 KB), and, 40 % of it, by the
// chains of waits around the pairs: so eight look-ups go out at once, the scans shift lanes instead
// of taking 18 barriers, and a wave reads four groups of sums before it decides (13.8 -> 12.6 ms at
// 160002; the atomics alone cost 0.4).  Whole graph call, two-pass bitmaps -> paged: N = 1000 0.31
// -> 0.23 ms, 18000 2.17 -> 1.60, 100000 (clustered) 17.3 -> 8.1, 160002 35.0 -> 12.7 (67 with hash
// sets, which it took there); rows of consecutive numbers, which share the rows they read, on one
// XCD: 5 % of it.  512 threads: 256 take 1.5 times, 1024 1.2 times as long at 160002.
struct X2Paged {
  int shift, pcap, cap, most;
};
constexpr int kPT = 512;

__device__ __forceinline__ int x2_page(int32_t* dir, int32_t* npages, int& spare, int pg,
                                       bool need) {
  // one lane of the wave per missing page takes a slot and publishes it; a slot lost to another
  // wave is the wave's next one (spare, the same in every lane).  No lane waits for another one.
  int sl = need ? *(volatile int32_t*)&dir[pg] : 0;
  unsigned long long open = __ballot(sl < 0);
  while (open) {
    const int leader = __ffsll((long long)open) - 1;
    const int lp = __shfl(pg, leader);
    int got = 0, left = spare;
    if ((int)(threadIdx.x & 63) == leader) {
      got = *(volatile int32_t*)&dir[lp];
      if (got < 0) {
        const int fresh = spare >= 0 ? spare : atomicAdd(npages, 1);
        const int old = atomicCAS(&dir[lp], -1, fresh);
        got = old < 0 ? fresh : old;
        left = old < 0 ? -1 : fresh;
      }
    }
    got = __shfl(got, leader);
    spare = __shfl(left, leader);
    if (sl < 0 && pg == lp) sl = got;
    open = __ballot(sl < 0);
  }
  return sl;
}

__global__ __launch_bounds__(kPT) void k_x2_rows_paged(
    const int32_t* __restrict__ hcol, const double* __restrict__ x0,
    const double* __restrict__ rbound, const int32_t* __restrict__ rlen, int n, int w, double tau,
    int all_ascending, X2Paged g, int32_t* __restrict__ cnt, int32_t* __restrict__ rows,
    int32_t* __restrict__ overflow) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t npages, seen;
  const int i = xcd_run(blockIdx.x, n);
  if (i >= n) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int NW = kPT / 64;
  const int ndir = ((n - 1) >> g.shift) + 1;
  const int flat = g.pcap << g.shift, ng = (flat + 63) >> 6;
  double* acc = reinterpret_cast<double*>(smem);
  double* xi = acc + flat;
  unsigned long long* kept = reinterpret_cast<unsigned long long*>(xi + w);
  int32_t* dir = reinterpret_cast<int32_t*>(kept + ng);
  int32_t* plist = dir + ndir;  // pages in use, ascending
  int32_t* ci = plist + g.pcap;
  int32_t* pre = ci + w;
  int32_t* red = pre + ng;  // kPT ints
  for (int t = threadIdx.x; t < w; t += kPT) {
    ci[t] = hcol[(int64_t)i * w + t];
    xi[t] = x0[(int64_t)i * w + t];
  }
  // a system of at most pcap pages gets them all, in order
  for (int q = threadIdx.x; q < ndir; q += kPT) dir[q] = ndir <= g.pcap ? q : -1;
  for (int q = threadIdx.x; q < flat; q += kPT) acc[q] = -0.0;
  if (threadIdx.x == 0) {
    seen = __hip_atomic_load(&overflow[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    npages = 0;
    red[0] = w;
  }
  __syncthreads();
  if (seen > g.most) {  // the same for the whole workgroup
    if (threadIdx.x == 0) cnt[i] = 0;
    return;
  }
  // the rows k of row i are its slots before the first padding entry
  for (int t = threadIdx.x; t < w; t += kPT)
    if ((unsigned)ci[t] >= (unsigned)n) atomicMin(&red[0], t);
  __syncthreads();
  const int kw = red[0];
  const int low = (1 << g.shift) - 1;
  int spare = -1;
  if (wave == 0) (void)x2_page(dir, &npages, spare, i >> g.shift, lane == 0);  // row i itself
  for (int t0 = wave; t0 < kw; t0 += 2 * NW) {  // two rows k at a time
    const int t1 = t0 + NW;
    const int k0 = ci[t0], k1 = t1 < kw ? ci[t1] : -1;
    const double a0 = xi[t0], a1 = t1 < kw ? xi[t1] : 0.0;
    const int l0 = rlen[k0], l1 = k1 >= 0 ? rlen[k1] : 0;
    const int64_t b0 = (int64_t)k0 * w, b1 = (int64_t)max(k1, 0) * w;
    for (int u0 = 0; u0 < max(l0, l1); u0 += 256) {
      int32_t j[8];
      double v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {  // every load of the batch first
        const int u = u0 + (q >> 1) * 64 + lane;
        const bool in = u < ((q & 1) ? l1 : l0);
        j[q] = in ? hcol[((q & 1) ? b1 : b0) + u] : -1;
        v[q] = in ? x0[((q & 1) ? b1 : b0) + u] : 0.0;
      }
      // every page's slot first, too: one wait for eight LDS reads; only a page not there yet (or
      // taken by another wave meanwhile) asks again
      int slot[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        slot[q] = (unsigned)j[q] < (unsigned)n ? *(volatile int32_t*)&dir[j[q] >> g.shift] : 0;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const bool ok = (unsigned)j[q] < (unsigned)n;
        if (__ballot(ok) == 0) continue;  // the same for the whole wave
        int sl = slot[q];
        if (__ballot(sl < 0)) sl = x2_page(dir, &npages, spare, ok ? j[q] >> g.shift : 0, ok);
        if (ok && sl < g.pcap)
          atomicAdd(&acc[(sl << g.shift) | (j[q] & low)], ((q & 1) ? a1 : a0) * v[q]);
      }
    }
  }
  __syncthreads();
  if (npages > g.pcap) {
    if (threadIdx.x == 0) {
      atomicMax(&overflow[0], npages);
      cnt[i] = 0;
    }
    return;
  }
  // the pages in use, ascending: each thread counts and then lists a run of the directory
  const int seg = (ndir + kPT - 1) / kPT;
  const int d0 = min((int)threadIdx.x * seg, ndir), d1 = min(d0 + seg, ndir);
  int mine = 0;
  for (int q = d0; q < d1; ++q) mine += dir[q] >= 0;
  int32_t used;
  int at = block_inclusive_scan<kPT>(mine, red, &used) - mine;
  // page and slot in a word: LDS holds neither 2^10 slots of 256 bytes nor a directory of 2^16
  // pages
  for (int q = d0; q < d1; ++q)
    if (dir[q] >= 0) plist[at++] = q << 10 | dir[q];
  __syncthreads();
  // decisions, 64 entries of the pages in ascending order per wave
  const double margin = x2_margin(kw, rbound[i], tau);
  const int total = used << g.shift, groups = (total + 63) >> 6;
  auto page_of = [&](int f) { return plist[f >> g.shift] >> 10; };
  constexpr int B = 4;  // groups whose sums a wave reads at once
  for (int qb = wave; qb < groups; qb += B * NW) {
    double sums[B];
    int cols[B];
#pragma unroll
    for (int e = 0; e < B; ++e) {
      const int f = ((qb + e * NW) << 6) | lane;
      const int pl = f < total ? plist[f >> g.shift] : 0;
      cols[e] = f < total ? (pl >> 10) << g.shift | (f & low) : n;
      sums[e] = f < total ? acc[(pl & 1023) << g.shift | (f & low)] : -0.0;
    }
#pragma unroll
    for (int e = 0; e < B; ++e) {
      const int q = qb + e * NW, j = cols[e];
      if (q >= groups) break;
      const double a = fabs(sums[e]);
      bool keep = j == i, band = false;
      if (j != i && j < n && !(sums[e] == 0.0 && signbit(sums[e]))) {
        band = all_ascending || fabs(a - tau) <= margin;
        keep = !band && a >= tau;
      }
      unsigned long long again = __ballot(band);
      while (again) {  // summed in ascending order, the whole wave on one entry
        const int l = __ffsll((long long)again) - 1;
        const double x = fabs(x2_sum_ascending(hcol, x0, ci, xi, kw, w, __shfl(j, l)));
        if (lane == l) keep = x >= tau;
        again &= again - 1;
      }
      const unsigned long long m = __ballot(keep);
      if (lane == 0) {
        kept[q] = m;
        pre[q] = __popcll(m);
      }
    }
  }
  __syncthreads();
  const int32_t nk = lds_exclusive_scan<kPT>(pre, groups, red);
  if (threadIdx.x == 0) cnt[i] = nk <= g.cap ? nk : 0;
  if (nk > g.cap) {
    if (threadIdx.x == 0) atomicMax(&overflow[1], nk);
    return;
  }
  int32_t* dst = rows + (int64_t)i * g.cap;
  for (int q = wave; q < groups; q += NW) {
    const unsigned long long m = kept[q];
    const int f = (q << 6) | lane;
    if ((m >> lane) & 1ull)
      dst[pre[q] + __popcll(m & ((1ull << lane) - 1ull))] =
          (page_of(f) << g.shift) | (f & low);
  }
}

size_t x2_paged_lds_bytes(int n, int w, const X2Paged& g) {
  const size_t flat = (size_t)g.pcap << g.shift, ng = (flat + 63) / 64;
  const size_t ndir = ((size_t)(n - 1) >> g.shift) + 1;
  return flat * 8 + (size_t)w * 8 + ng * 8 + ndir * 4 + (size_t)g.pcap * 4 + (size_t)w * 4 +
         ng * 4 + (size_t)kPT * 4 + 64;
}

size_t x2_hash_lds_bytes(int w, int cap, int log2h, int log2u) {
  return (size_t)cap * 8 + (size_t)w * 8 + ((size_t)2 << log2h) * 4 + ((size_t)1 << log2u) * 4 +
         (size_t)w * 4 + (size_t)kT * 4 + 64;
}

// row i of the staging array (cnt[i] columns at i * cap) -> the CSR at row_ptr[i]
__global__ __launch_bounds__(kT) void k_x2_compact(const int32_t* __restrict__ rows, int cap,
                                                   const int32_t* __restrict__ cnt,
                                                   const int32_t* __restrict__ row_ptr,
                                                   int32_t* __restrict__ out_col) {
  const int i = blockIdx.x;
  const int32_t* src = rows + (int64_t)i * cap;
  int32_t* dst = out_col + row_ptr[i];
  for (int t = threadIdx.x; t < cnt[i]; t += kT) dst[t] = src[t];
}

size_t x2_lds_bytes(int n, int w, int cap) {
  const int nw = (n + 31) >> 5;
  return (size_t)cap * 8 + (size_t)w * 8 + (size_t)nw * 4 + (size_t)(nw + 1) * 4 + (size_t)w * 4 +
         (size_t)kT * 4 + 64;
}

// ---- row unions through an LDS bitmap (pattern graphs, symmetrisation) --------------------
// Row i of the result = (row i of up to three CSR inputs) U {i}, sorted and unique.
template <int PASS>
__global__ __launch_bounds__(kT) void k_union_rows(int n, const int32_t* __restrict__ rp0,
                                                   const int32_t* __restrict__ c0,
                                                   const int32_t* __restrict__ rp1,
                                                   const int32_t* __restrict__ c1,
                                                   const int32_t* __restrict__ rp2,
                                                   const int32_t* __restrict__ c2,
                                                   int32_t* __restrict__ cnt,
                                                   const int32_t* __restrict__ row_ptr,
                                                   int32_t* __restrict__ out_col) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int i = blockIdx.x;
  const int nw = (n + 31) >> 5;
  uint32_t* bits = reinterpret_cast<uint32_t*>(smem);
  int32_t* wc = reinterpret_cast<int32_t*>(bits + nw);
  int32_t* red = wc + nw;
  for (int q = threadIdx.x; q < nw; q += kT) bits[q] = 0u;
  __syncthreads();
  for (int p = rp0[i] + threadIdx.x; p < rp0[i + 1]; p += kT) {
    const int j = c0[p];
    atomicOr(&bits[j >> 5], 1u << (j & 31));
  }
  if (rp1)
    for (int p = rp1[i] + threadIdx.x; p < rp1[i + 1]; p += kT) {
      const int j = c1[p];
      atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
  if (rp2)
    for (int p = rp2[i] + threadIdx.x; p < rp2[i + 1]; p += kT) {
      const int j = c2[p];
      atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
  if (threadIdx.x == 0) atomicOr(&bits[i >> 5], 1u << (i & 31));
  __syncthreads();
  for (int q = threadIdx.x; q < nw; q += kT) wc[q] = __popc(bits[q]);
  __syncthreads();
  const int32_t tot = lds_exclusive_scan<kT>(wc, nw, red);
  if (PASS == 0) {
    if (threadIdx.x == 0) cnt[i] = tot;
    return;
  }
  const int32_t base = row_ptr[i];
  for (int q = threadIdx.x; q < nw; q += kT) {
    uint32_t word = bits[q];
    int32_t pos = base + wc[q];
    while (word) {
      const int b = __ffs(word) - 1;
      out_col[pos++] = (q << 5) + b;
      word &= word - 1u;
    }
  }
}


// two-hop closure: row i of the result = union over k in row i of P of row k of P (paths of
// length two; P contains every self-loop, so one-hop edges are included), sorted, unique
template <int PASS>
__global__ __launch_bounds__(kT) void k_twohop_rows(int n, const int32_t* __restrict__ rp,
                                                    const int32_t* __restrict__ c,
                                                    int32_t* __restrict__ cnt,
                                                    const int32_t* __restrict__ row_ptr,
                                                    int32_t* __restrict__ out_col) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int i = blockIdx.x;
  const int nw = (n + 31) >> 5;
  uint32_t* bits = reinterpret_cast<uint32_t*>(smem);
  int32_t* wc = reinterpret_cast<int32_t*>(bits + nw);
  int32_t* red = wc + nw;
  for (int q = threadIdx.x; q < nw; q += kT) bits[q] = 0u;
  __syncthreads();
  for (int a = rp[i]; a < rp[i + 1]; ++a) {
    const int k = c[a];
    for (int p = rp[k] + threadIdx.x; p < rp[k + 1]; p += kT) {
      const int j = c[p];
      atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
  }
  if (threadIdx.x == 0) atomicOr(&bits[i >> 5], 1u << (i & 31));
  __syncthreads();
  for (int q = threadIdx.x; q < nw; q += kT) wc[q] = __popc(bits[q]);
  __syncthreads();
  const int32_t tot = lds_exclusive_scan<kT>(wc, nw, red);
  if (PASS == 0) {
    if (threadIdx.x == 0) cnt[i] = tot;
    return;
  }
  const int32_t base = row_ptr[i];
  for (int q = threadIdx.x; q < nw; q += kT) {
    uint32_t word = bits[q];
    int32_t pos = base + wc[q];
    while (word) {
      const int b = __ffs(word) - 1;
      out_col[pos++] = (q << 5) + b;
      word &= word - 1u;
    }
  }
}

// entries of an ELL matrix with |a| >= tau, as (row-list) CSR counts / fill, in slot order (ELL
// rows are ascending, so the output rows are); a row ends at its first padding entry.  One wave
// per row, 64 slots at a time: a previous D is some 2000 slots wide and its rows are read twice,
// so what counts is that the reads are coalesced (a thread per row: 1.34 + 1.03 ms at N = 4096 x
// 2304, this way 0.024 + 0.016).
template <int PASS>
__global__ __launch_bounds__(kT) void k_ell_threshold(const int32_t* __restrict__ col,
                                                      const double* __restrict__ val, int n, int w,
                                                      double tau, int32_t* __restrict__ cnt,
                                                      const int32_t* __restrict__ row_ptr,
                                                      int32_t* __restrict__ out) {
  const int i = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  const int64_t base = (int64_t)i * w;
  int pos = PASS ? row_ptr[i] : 0;
  for (int t0 = 0; t0 < w; t0 += 64) {
    const int t = t0 + lane;
    const int32_t j = t < w ? col[base + t] : -1;
    const double a = t < w ? val[base + t] : 0.0;
    const unsigned long long end = __ballot(j < 0);
    const bool before = end == 0 || lane < __ffsll((long long)end) - 1;
    const bool keep = before && (unsigned)j < (unsigned)n && fabs(a) >= tau;
    const unsigned long long m = __ballot(keep);
    if (PASS && keep) out[pos + __popcll(m & ((1ull << lane) - 1ull))] = j;
    pos += __popcll(m);
    if (end) break;
  }
  if (!PASS && lane == 0) cnt[i] = pos;
}

// transpose of a CSR pattern: count per column, then fill (order within a row arbitrary); a wave
// per row
__global__ __launch_bounds__(kT) void k_tr_count(const int32_t* __restrict__ rp,
                                                 const int32_t* __restrict__ c, int n,
                                                 int32_t* __restrict__ cnt) {
  const int i = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  for (int p = rp[i] + lane; p < rp[i + 1]; p += 64) atomicAdd(&cnt[c[p]], 1);
}
__global__ __launch_bounds__(kT) void k_tr_fill(const int32_t* __restrict__ rp,
                                                const int32_t* __restrict__ c, int n,
                                                const int32_t* __restrict__ trp,
                                                int32_t* __restrict__ fill,
                                                int32_t* __restrict__ tc) {
  const int i = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  for (int p = rp[i] + lane; p < rp[i + 1]; p += 64) {
    const int j = c[p];
    tc[trp[j] + atomicAdd(&fill[j], 1)] = i;
  }
}

__global__ void k_zero_i32(int32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---- RCUT graph (divide-and-conquer comparison): sites within r_cut, periodic cube ----------
// Site a's neighbours b (ascending, a itself included) with the canonical minimum-image squared
// distance below rc2.  PASS 0 counts per site; PASS 1 writes the orbital rows of site a in
// ascending column order (a block-wide scan over each 256-site window keeps the order).
template <int PASS>
__global__ __launch_bounds__(kT) void k_rcut_rows(const double* __restrict__ pos, int n_sites,
                                                  int m, double box, double rc2,
                                                  int32_t* __restrict__ cnt,
                                                  const int32_t* __restrict__ row_ptr,
                                                  int32_t* __restrict__ col) {
  __shared__ int32_t scan[kT];
  __shared__ int32_t base;
  const int a = blockIdx.x;
  const double xa = pos[3 * a], ya = pos[3 * a + 1], za = pos[3 * a + 2];
  if (threadIdx.x == 0) base = 0;
  __syncthreads();
  for (int b0 = 0; b0 < n_sites; b0 += kT) {
    const int b = b0 + threadIdx.x;
    int hit = 0;
    if (b < n_sites) {
      double dx = pos[3 * b] - xa, dy = pos[3 * b + 1] - ya, dz = pos[3 * b + 2] - za;
      dx = dx - box * rint(dx / box);
      dy = dy - box * rint(dy / box);
      dz = dz - box * rint(dz / box);
      const double r2 = (dx * dx + dy * dy) + dz * dz;
      hit = r2 < rc2 ? 1 : 0;
    }
    scan[threadIdx.x] = hit;
    __syncthreads();
    for (int h = 1; h < kT; h <<= 1) {  // inclusive scan (Hillis-Steele)
      const int v = threadIdx.x >= h ? scan[threadIdx.x - h] : 0;
      __syncthreads();
      scan[threadIdx.x] += v;
      __syncthreads();
    }
    if (PASS == 1 && hit) {
      const int rank = base + scan[threadIdx.x] - 1;  // neighbour index of b in site a's list
      for (int o = 0; o < m; ++o) {
        int32_t* out = col + row_ptr[a * m + o];
        for (int q = 0; q < m; ++q) out[rank * m + q] = b * m + q;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) base += scan[kT - 1];
    __syncthreads();
  }
  if (PASS == 0 && threadIdx.x == 0)
    for (int o = 0; o < m; ++o) cnt[a * m + o] = base * m;
}

int blocks_for(int64_t n, int t) { return (int)((n + t - 1) / t); }

void check_lds(size_t bytes, const char* what) {
  if (bytes > 160 * 1024)
    fail(GB_EUNSUPPORTED, "%s needs %zu bytes of LDS per workgroup (limit 163840)", what, bytes);
}

// union of one to three CSRs plus self-loops -> out (sorted rows)
void union_rows(int n, const int32_t* rp0, const int32_t* c0, const int32_t* rp1,
                const int32_t* c1, const int32_t* rp2, const int32_t* c2, Csr& out,
                hipStream_t s) {
  const int nw = (n + 31) >> 5;
  const size_t lds = (size_t)nw * 8 + kT * 4 + 64;
  check_lds(lds, "graph row union");
  DBuf<int32_t> cnt(n, s);
  out.n = n;
  out.row_ptr = DBuf<int32_t>(n + 1, s);
  hipLaunchKernelGGL(k_union_rows<0>, dim3(n), dim3(kT), lds, s, n, rp0, c0, rp1, c1, rp2, c2,
                     cnt.get(), nullptr, nullptr);
  GB_LAUNCH_CHECK();
  exclusive_scan_i32(cnt.get(), out.row_ptr.get(), n, s);
  int32_t nnz = 0;
  GB_HIP(hipMemcpyAsync(&nnz, out.row_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
  GB_HIP(hipStreamSynchronize(s));
  out.nnz = nnz;
  out.col = DBuf<int32_t>(nnz, s);
  hipLaunchKernelGGL(k_union_rows<1>, dim3(n), dim3(kT), lds, s, n, rp0, c0, rp1, c1, rp2, c2,
                     nullptr, out.row_ptr.get(), out.col.get());
  GB_LAUNCH_CHECK();
}

// CSR of the entries |a| >= tau of an ELL matrix (row-wise, rows ascending)
void ell_threshold(const gb_ell& A, double tau, DBuf<int32_t>& rp, DBuf<int32_t>& c,
                   int32_t& nnz, hipStream_t s) {
  const int n = A.n;
  DBuf<int32_t> cnt(n, s);
  rp = DBuf<int32_t>(n + 1, s);
  hipLaunchKernelGGL(k_ell_threshold<0>, dim3(blocks_for(n, kT / 64)), dim3(kT), 0, s, A.col, A.val,
                     n, A.width, tau, cnt.get(), nullptr, nullptr);
  GB_LAUNCH_CHECK();
  exclusive_scan_i32(cnt.get(), rp.get(), n, s);
  nnz = 0;
  GB_HIP(hipMemcpyAsync(&nnz, rp.get() + n, 4, hipMemcpyDeviceToHost, s));
  GB_HIP(hipStreamSynchronize(s));
  c = DBuf<int32_t>(nnz > 0 ? nnz : 1, s);
  hipLaunchKernelGGL(k_ell_threshold<1>, dim3(blocks_for(n, kT / 64)), dim3(kT), 0, s, A.col, A.val,
                     n, A.width, tau, nullptr, rp.get(), c.get());
  GB_LAUNCH_CHECK();
}

void transpose(int n, const int32_t* rp, const int32_t* c, int64_t nnz, DBuf<int32_t>& trp,
               DBuf<int32_t>& tc, hipStream_t s) {
  DBuf<int32_t> cnt(n, s), fill(n, s);
  hipLaunchKernelGGL(k_zero_i32, dim3(blocks_for(n, kT)), dim3(kT), 0, s, cnt.get(), (int64_t)n);
  hipLaunchKernelGGL(k_zero_i32, dim3(blocks_for(n, kT)), dim3(kT), 0, s, fill.get(), (int64_t)n);
  GB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_tr_count, dim3(blocks_for(n, kT / 64)), dim3(kT), 0, s, rp, c, n, cnt.get());
  GB_LAUNCH_CHECK();
  trp = DBuf<int32_t>(n + 1, s);
  exclusive_scan_i32(cnt.get(), trp.get(), n, s);
  tc = DBuf<int32_t>(nnz > 0 ? nnz : 1, s);
  hipLaunchKernelGGL(k_tr_fill, dim3(blocks_for(n, kT / 64)), dim3(kT), 0, s, rp, c, n, trp.get(),
                     fill.get(), tc.get());
  GB_LAUNCH_CHECK();
}

}  // namespace

static bool vertex_sets_forced() {
  const char* e = std::getenv("GB_VERTEX_SETS");
  return e && (std::string(e) == "hash" || std::string(e) == "bitmap");
}

bool use_hash_sets(int n, int from) {
  const char* e = std::getenv("GB_VERTEX_SETS");
  if (e && std::string(e) == "hash") return true;
  if (e && std::string(e) == "bitmap") return false;
  return n > from;
}

// part: 3 nb partials, then the result
void bounds_into(const gb_ell& H, hipStream_t s, double* part, int nb, double* emin,
                 double* emax) {
  hipLaunchKernelGGL(k_disc_partials, dim3(nb), dim3(kT), 0, s, H.col, H.val, H.n, H.width, part);
  GB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_disc_final, dim3(1), dim3(kT), 0, s, part, nb, part + 3 * nb);
  GB_LAUNCH_CHECK();
  double h[3];
  GB_HIP(hipMemcpyAsync(h, part + 3 * nb, sizeof(h), hipMemcpyDeviceToHost, s));
  GB_HIP(hipStreamSynchronize(s));
  if (h[2] != 0.0)
    fail(GB_EINVAL, "H holds NaN or Inf values (%.0f rows): no spectral bounds", h[2]);
  *emin = h[0];
  *emax = h[1];
}

int disc_blocks(int n) { return std::min(blocks_for(n, kDiscGroup), kNoallocBlocks); }

void bounds(const gb_ell& H, hipStream_t s, double* emin, double* emax) {
  const int nb = disc_blocks(H.n);
  DBuf<double> part(3 * (size_t)nb + 3, s);
  bounds_into(H, s, part.get(), nb, emin, emax);
}

// Device address of `scratch` on the current device, looked up once per device (each GPU holds
// its own copy of the array).  Host code uses only this address, never the array's name.
double* scratch_ptr() {
  static std::mutex mu;
  static std::map<int, double*> ptrs;
  int dev = 0;
  GB_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(mu);
  auto it = ptrs.find(dev);
  if (it != ptrs.end()) return it->second;
  void* p = nullptr;
  GB_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
  if (!p) fail(GB_EHIP, "no device address for the bounds scratch array");
  ptrs[dev] = static_cast<double*>(p);
  return static_cast<double*>(p);
}

void bounds_noalloc(const gb_ell& H, hipStream_t s, double* emin, double* emax) {
  bounds_into(H, s, scratch_ptr(), disc_blocks(H.n), emin, emax);
}

void x0_ell(const gb_ell& H, double emin, double emax, double* x0, hipStream_t s) {
  const int64_t tot = (int64_t)H.n * H.width;
  const double denom = emax - emin;
  hipLaunchKernelGGL(k_x0, dim3(blocks_for(tot, kT)), dim3(kT), 0, s, H.col, H.val, H.n, H.width,
                     emax, denom, x0);
  GB_LAUNCH_CHECK();
}

// the bounds b_i of the X2 kernels' order-free sums (see k_x2_rows)
// and the rows' lengths
void x2_row_bounds(const gb_ell& H, const double* x0, DBuf<double>& rb, DBuf<int32_t>& rlen,
                   hipStream_t s) {
  const int n = H.n, w = H.width;
  DBuf<double> amax(n, s);
  rb = DBuf<double>(n, s);
  rlen = DBuf<int32_t>(n, s);
  const int nb = blocks_for(n, kT / 64);
  hipLaunchKernelGGL(k_row_absmax, dim3(nb), dim3(kT), 0, s, H.col, x0, n, w, amax.get(),
                     rlen.get());
  GB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_x2_bound, dim3(nb), dim3(kT), 0, s, H.col, x0, amax.get(), n, w,
                     rb.get());
  GB_LAUNCH_CHECK();
}

// GB_X2_SUMS=ascending: every candidate is summed again in ascending order (a check of the
// path that the candidates near tau take)
int x2_all_ascending() {
  const char* e = std::getenv("GB_X2_SUMS");
  return e && std::string(e) == "ascending" ? 1 : 0;
}

// X2 graph through k_x2_rows_paged; false when its pages do not fit (vertices numbered without
// regard to place, very long rows), which leaves the row sets to the two-pass kernels.  Page
// edge: the directory grows with n / 2^shift and the pages a row touches shrink with 2^shift.
bool graph_x2_paged(const gb_ell& H, const double* x0, double tau, Csr& out, hipStream_t s) {
  const int n = H.n, w = H.width;
  X2Paged g;
  g.shift = n <= (1 << 16) ? 5 : n <= (1 << 18) ? 6 : n <= (1 << 20) ? 7 : 8;
  const int ndir = ((n - 1) >> g.shift) + 1;
  g.pcap = std::min(ndir, g.shift == 5 ? 192 : g.shift == 6 ? 104 : 64);
  g.cap = std::min(n, 2048);
  const size_t most = 158 * 1024;
  if (x2_paged_lds_bytes(n, w, g) > most) return false;
  // Rows that ask for more pages: a second attempt costs as much as the first and has fewer
  // workgroups per CU.  Bitmaps take less (randomly numbered, N = 8000, 239 slots: 1.8 ms for both
  // attempts, 0.9 for bitmaps; N = 150000, 61 slots: 18.3 and 6.3); hash sets, which take their
  // place above 3 << 16, do not (21.4).
  const bool again = n > 3 << 16;
  g.most = g.pcap;
  if (again) {
    X2Paged full = g;
    while (g.most < ndir && (full.pcap = g.most + 1, x2_paged_lds_bytes(n, w, full) <= most))
      ++g.most;
  }
  DBuf<int32_t> cnt(n, s), ovf(2, s), rows, rlen;
  DBuf<double> rb;
  x2_row_bounds(H, x0, rb, rlen, s);
  const int all_asc = x2_all_ascending();
  out.n = n;
  out.row_ptr = DBuf<int32_t>(n + 1, s);
  int32_t h[3] = {0, 0, 0};
  for (int attempt = 0;; ++attempt) {
    rows = DBuf<int32_t>((size_t)n * g.cap, s);
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, s, ovf.get(), (int64_t)2);
    hipLaunchKernelGGL(k_x2_rows_paged, dim3(xcd_grid(n)), dim3(kPT),
                       x2_paged_lds_bytes(n, w, g), s, H.col, x0, rb.get(), rlen.get(), n, w, tau, all_asc, g, cnt.get(), rows.get(),
                       ovf.get());
    GB_LAUNCH_CHECK();
    exclusive_scan_i32(cnt.get(), out.row_ptr.get(), n, s);
    GB_HIP(hipMemcpyAsync(&h[0], out.row_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
    GB_HIP(hipMemcpyAsync(&h[1], ovf.get(), 8, hipMemcpyDeviceToHost, s));
    GB_HIP(hipStreamSynchronize(s));
    if (h[1] == 0 && h[2] == 0) break;
    // more pages (a row whose pages ran out has not counted what it keeps), more kept entries
    if (attempt == 3 || h[1] > g.most) return false;
    if (h[1] > 0) g.pcap = std::min(g.most, h[1] + h[1] / 8);
    if (h[2] > 0) g.cap = std::min(n, (h[2] + 255) / 256 * 256);
    if (x2_paged_lds_bytes(n, w, g) > most) return false;
  }
  out.nnz = h[0];
  out.col = DBuf<int32_t>(h[0] > 0 ? h[0] : 1, s);
  hipLaunchKernelGGL(k_x2_compact, dim3(n), dim3(kT), 0, s, rows.get(), g.cap, cnt.get(),
                     out.row_ptr.get(), out.col.get());
  GB_LAUNCH_CHECK();
  return true;
}

// X2 graph through the hash-set kernel: candidate capacity 2048 to start with (two workgroups
// per CU), raised to the largest count a row reports and run again (at most twice).
void graph_x2_hash(const gb_ell& H, const double* x0, double tau, Csr& out, hipStream_t s) {
  const int n = H.n, w = H.width;
  int cap = (int)std::min<int64_t>(std::min<int64_t>((int64_t)w * w, n) + 1, 2048);
  cap = std::max(cap, kT);
  DBuf<int32_t> cnt(n, s), ovf(1, s), rows, rlen;
  DBuf<double> rb;
  x2_row_bounds(H, x0, rb, rlen, s);
  const int all_asc = x2_all_ascending();
  out.n = n;
  out.row_ptr = DBuf<int32_t>(n + 1, s);
  int32_t h[2] = {0, 0};
  for (int attempt = 0;; ++attempt) {
    const int log2h = ceil_log2((int64_t)cap + kT + 1), log2u = ceil_log2(cap);
    const size_t lds = x2_hash_lds_bytes(w, cap, log2h, log2u);
    if (lds > 160 * 1024)
      fail(GB_EUNSUPPORTED, "X2 graph: a row has %d two-hop candidates, more than LDS holds", cap);
    rows = DBuf<int32_t>((size_t)n * cap, s);
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, s, ovf.get(), (int64_t)1);
    hipLaunchKernelGGL(k_x2_rows_hash, dim3(n), dim3(kT), lds, s, H.col, x0, rb.get(), n, w,
                       1.0f / (float)w, tau, all_asc, cap, log2h, log2u, cnt.get(), rows.get(),
                       ovf.get());
    GB_LAUNCH_CHECK();
    exclusive_scan_i32(cnt.get(), out.row_ptr.get(), n, s);
    GB_HIP(hipMemcpyAsync(&h[0], out.row_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
    GB_HIP(hipMemcpyAsync(&h[1], ovf.get(), 4, hipMemcpyDeviceToHost, s));
    GB_HIP(hipStreamSynchronize(s));
    if (h[1] == 0) break;
    if (attempt == 2) fail(GB_EUNSUPPORTED, "X2 graph: candidate count did not settle");
    // a stopped row counted at least cap + 1 candidates; grow past what was reported
    cap = std::max(((h[1] + 255) / 256) * 256, 2 * cap);
  }
  out.nnz = h[0];
  out.col = DBuf<int32_t>(h[0] > 0 ? h[0] : 1, s);
  hipLaunchKernelGGL(k_x2_compact, dim3(n), dim3(kT), 0, s, rows.get(), cap, cnt.get(),
                     out.row_ptr.get(), out.col.get());
  GB_LAUNCH_CHECK();
}

// Does one pass with paged accumulators beat two passes over candidate sets?  It saves a visit of
// every pair, and bitmaps whose handling grows with n, but gives pages out row by row and clears
// and reads them whole, which takes rows of many pairs, the more so the further a row's partners
// are apart in number.  Measured, one pass / two (ms), w the ELL width, on places in Morton order
// (m) and lattices in row order (l), which spread a row over more pages:
//   n = 4096      w  62  0.213 / 0.189 m    w 121  0.253 / 0.278 m    w 247  0.359 / 0.625 m
//   n = 8192      w 123  0.475 / 0.386 m    w  54  0.364 / 0.229 l    w 241  0.817 / 1.03 m
//   n = 18000     w 165  1.03 / 1.00 m      w  73  0.611 / 0.412 m    w 253  1.88 / 2.47 m
//   n = 32768     w 131  1.67 / 1.53 m      w 125  2.11 / 1.68 l      w 255  3.22 / 4.45 m
//   n = 64000     w  77  1.97 / 1.81 m      w 125  4.35 / 3.20 l      w 257  5.63 / 8.79 m
//   n = 80000     w  77  2.20 / 2.10 m      w  27  1.91 / 1.04 l      w 137  3.51 / 3.89 m
//   n = 100000    w  41  1.74 / 1.82 m      w  81  2.94 / 3.46 m      w 263  8.28 / 15.8 m
//   n = 125000    w   7  1.92 / 3.22 l      w  27  2.67 / 3.47 l      w 255  10.6 / 21.8 m
// Above 2^17 two passes use hash sets, whose cost does not grow with n: narrow rows stay with them
// (n = 166375, w 7: 2.64 / 1.32 l; n = 512000, w 27: 22.5 / 11.4 l), the others do not (n = 150000,
// w 41: 2.87 / 10.7 m; n = 262144, w 125: 18.8 / 57.8 l).
bool x2_paged_pays(int n, int w) {
  const int least = n <= 4096 ? 96 : n <= 65536 ? 192 : n <= 98304 ? 128 : n <= 114688 ? 64
                  : n <= (1 << 17) ? 1 : 32;
  return w >= least;
}

void graph_x2(const gb_ell& H, const double* x0, double tau, Csr& out, hipStream_t s) {
  const int n = H.n, w = H.width;
  // what the two-pass kernels' rows hold, whichever kernels would take these
  if (w > kX2Q * kT) fail(GB_EUNSUPPORTED, "X2 graph: ELL width %d above %d", w, kX2Q * kT);
  // tau = 0 keeps candidates whose sum is 0, which only the candidate sets know
  if (tau > 0.0 && !vertex_sets_forced() && x2_paged_pays(n, w) &&
      graph_x2_paged(H, x0, tau, out, s))
    return;
  // two passes, bitmaps against hash sets: 37 / 67 ms at n = 160002 (w 255), 125 / 112 at n =
  // 262000; rows below 32 slots 3.2 / 1.3 (w 7) and 3.9 / 3.9 (w 27) at n = 166375
  if (use_hash_sets(n, w < 32 ? 1 << 17 : 3 << 16)) {
    graph_x2_hash(H, x0, tau, out, s);
    return;
  }
  // candidate capacity: small enough for six or more workgroups per CU at n up to ~2e4 (the
  // accumulators are most of the LDS); a row with more two-hop candidates makes the launch
  // report its count, and the launch reruns with it
  const size_t fixed = x2_lds_bytes(n, w, 0);
  if (fixed > 150 * 1024) fail(GB_EUNSUPPORTED, "X2 graph: n = %d too large for one LDS bitmap", n);
  const int64_t cap_lds = (int64_t)((160 * 1024 - fixed) / 8);
  int64_t cap = std::min<int64_t>(std::min<int64_t>((int64_t)w * w, n), 2048);
  cap = std::min(cap, cap_lds);
  DBuf<int32_t> cnt(n, s), ovf(1, s), rows, rlen;
  DBuf<double> rb;
  x2_row_bounds(H, x0, rb, rlen, s);
  const int all_asc = x2_all_ascending();
  out.n = n;
  out.row_ptr = DBuf<int32_t>(n + 1, s);
  int32_t h[2];
  for (int attempt = 0; attempt < 2; ++attempt) {
    const size_t lds = x2_lds_bytes(n, w, (int)cap);
    check_lds(lds, "X2 graph");
    rows = DBuf<int32_t>((size_t)n * cap, s);
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, s, ovf.get(), (int64_t)1);
    hipLaunchKernelGGL(k_x2_rows, dim3(n), dim3(kT), lds, s, H.col, x0, rb.get(), n, w,
                       1.0f / (float)w, tau, all_asc, (int)cap, cnt.get(), rows.get(), ovf.get());
    GB_LAUNCH_CHECK();
    exclusive_scan_i32(cnt.get(), out.row_ptr.get(), n, s);
    GB_HIP(hipMemcpyAsync(&h[0], out.row_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
    GB_HIP(hipMemcpyAsync(&h[1], ovf.get(), 4, hipMemcpyDeviceToHost, s));
    GB_HIP(hipStreamSynchronize(s));
    if (h[1] == 0) break;
    if (attempt == 1 || h[1] > cap_lds)
      fail(GB_EUNSUPPORTED, "X2 graph: a row has %d two-hop candidates, LDS capacity is %lld",
           h[1], (long long)cap_lds);
    cap = ((h[1] + 255) / 256) * 256;
    cap = std::min(cap, cap_lds);
  }
  out.nnz = h[0];
  out.col = DBuf<int32_t>(h[0] > 0 ? h[0] : 1, s);
  hipLaunchKernelGGL(k_x2_compact, dim3(n), dim3(kT), 0, s, rows.get(), (int)cap, cnt.get(),
                     out.row_ptr.get(), out.col.get());
  GB_LAUNCH_CHECK();
}

void graph_pattern(const gb_ell& A, double tau, Csr& out, hipStream_t s) {
  DBuf<int32_t> rp, c, trp, tc;
  int32_t nnz = 0;
  ell_threshold(A, tau, rp, c, nnz, s);
  transpose(A.n, rp.get(), c.get(), nnz, trp, tc, s);
  union_rows(A.n, rp.get(), c.get(), trp.get(), tc.get(), nullptr, nullptr, out, s);
}

void graph_rcut(const double* pos, int n_sites, int m, double box, double r_cut, Csr& out,
                hipStream_t s) {
  const int n = n_sites * m;
  DBuf<int32_t> cnt(n, s);
  out.n = n;
  out.row_ptr = DBuf<int32_t>(n + 1, s);
  const double rc2 = r_cut * r_cut;
  hipLaunchKernelGGL(k_rcut_rows<0>, dim3(n_sites), dim3(kT), 0, s, pos, n_sites, m, box, rc2,
                     cnt.get(), nullptr, nullptr);
  GB_LAUNCH_CHECK();
  exclusive_scan_i32(cnt.get(), out.row_ptr.get(), n, s);
  int32_t nnz = 0;
  GB_HIP(hipMemcpyAsync(&nnz, out.row_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
  GB_HIP(hipStreamSynchronize(s));
  out.nnz = nnz;
  out.col = DBuf<int32_t>(nnz > 0 ? nnz : 1, s);
  hipLaunchKernelGGL(k_rcut_rows<1>, dim3(n_sites), dim3(kT), 0, s, pos, n_sites, m, box, rc2,
                     nullptr, out.row_ptr.get(), out.col.get());
  GB_LAUNCH_CHECK();
}

void graph_dprev_symbolic(const gb_ell& H, const gb_ell& Dp, double tau_d, Csr& out,
                          hipStream_t s) {
  // P = pattern(H) U {|D_prev| >= tau_d} U its transpose (symmetric, with self-loops), then
  // the symbolic square: Eq. 8 with eps = 0
  Csr hp, P;
  graph_pattern(H, 0.0, hp, s);
  graph_union_dprev(hp, Dp, tau_d, P, s);
  const int n = H.n;
  const int nw = (n + 31) >> 5;
  const size_t lds = (size_t)nw * 8 + kT * 4 + 64;
  check_lds(lds, "two-hop graph");
  DBuf<int32_t> cnt(n, s);
  out.n = n;
  out.row_ptr = DBuf<int32_t>(n + 1, s);
  hipLaunchKernelGGL(k_twohop_rows<0>, dim3(n), dim3(kT), lds, s, n, P.row_ptr.get(), P.col.get(),
                     cnt.get(), nullptr, nullptr);
  GB_LAUNCH_CHECK();
  exclusive_scan_i32(cnt.get(), out.row_ptr.get(), n, s);
  int32_t nnz = 0;
  GB_HIP(hipMemcpyAsync(&nnz, out.row_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
  GB_HIP(hipStreamSynchronize(s));
  out.nnz = nnz;
  out.col = DBuf<int32_t>(nnz > 0 ? nnz : 1, s);
  hipLaunchKernelGGL(k_twohop_rows<1>, dim3(n), dim3(kT), lds, s, n, P.row_ptr.get(), P.col.get(),
                     nullptr, out.row_ptr.get(), out.col.get());
  GB_LAUNCH_CHECK();
}

void graph_union_dprev(const Csr& base, const gb_ell& Dp, double tau_d, Csr& out,
                       hipStream_t s) {
  // column-ELL row i lists the rows r of column i with |D_ri| >= tau_d: edges (r, i).
  // The union of base (symmetric), that list (row i gets r) and its transpose (row r gets i)
  // is symmetric.
  DBuf<int32_t> rp, c, trp, tc;
  int32_t nnz = 0;
  ell_threshold(Dp, tau_d, rp, c, nnz, s);
  transpose(Dp.n, rp.get(), c.get(), nnz, trp, tc, s);
  union_rows(Dp.n, base.row_ptr.get(), base.col.get(), rp.get(), c.get(), trp.get(), tc.get(),
             out, s);
}

}  // namespace gbi
