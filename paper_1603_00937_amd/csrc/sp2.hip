// Batched SP2 on the subgraph blocks: gather, the MFMA squaring kernel, the FP64 trace /
// branch decision, the update, refinement, the column scatter into D and the final checks.
//
// Data layout in HBM: every subgraph s owns a dense row-major block of npad_s x npad_s
// elements (npad_s = n_s rounded up to 64) at element offset off_s of one batch buffer; the
// padding rows and columns are zero and stay zero under X^2 and 2X - X^2.  Two (three with
// refinement) such buffers ping-pong.  Core vertices are the first k_s rows of each block.
#include "internal.h"

#include <chrono>
#include <cmath>
#include <cstring>
#include <cstdlib>
#include <functional>
#include <string>
#include <map>
#include <mutex>
#include <numeric>
#include <thread>
#include <type_traits>

#pragma clang fp contract(off)

namespace gbi {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
  using acc_t = d4v;
  static constexpr int KC = 16;  // k elements per 128-byte row chunk
  __device__ static acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // output register r of lane l holds row (4r + l/16), column l%16 of the 16x16 block
  __device__ static int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
template <>
struct Mfma<float> {
  using acc_t = f4v;
  static constexpr int KC = 32;
  __device__ static acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // output register r of lane l holds row (4(l/16) + r), column l%16
  __device__ static int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

typedef __attribute__((address_space(3))) void lds_void;

// Target builtins are called only from these non-template device functions: a kernel template
// that names one directly is dropped from the host pass (no launch stub is emitted for it).
// 16-byte global -> LDS copy of one lane: lane L of the wave fills bytes [16L, 16L + 16) of
// the 1-KB LDS window that starts at `lds` (the same for every lane of the wave).
__device__ inline void load_lds16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, (lds_void*)lds, 16, 0, 0);
}
__device__ inline f4v mma_bf16(bf8v a, bf8v b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
// fp16 planes travel in the same 16-byte registers as bf16 ones and are reinterpreted here
__device__ inline f4v mma_f16(bf8v a, bf8v b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8v, a),
                                                __builtin_bit_cast(h8v, b), c, 0, 0, 0);
}
// plane products of either type
template <bool F16>
__device__ __forceinline__ f4v mma_p(bf8v a, bf8v b, f4v c) {
  if constexpr (F16) return mma_f16(a, b, c);
  else return mma_bf16(a, b, c);
}


namespace {

constexpr int kT = 256;
constexpr int kBT = 128;  // workgroup tile edge

// A block of n rows is stored as padded(n) rows of as many values, zero beyond n.  The squares'
// tiles carry n: the sums over k end with the chunk that holds row n - 1, and a wave whose block
// begins beyond it only writes its zeros, so the padding (3 % of the rows at 900, half a percent
// at 5000) is stored but not multiplied; the sums are the same without its zeros.  Step at N =
// 1024 (64 FP64 blocks of ~900 rows) 20.68 -> 20.38 ms, FP32 density at N = 3000 46.29 -> 45.77;
// the 16-bit squares, which the power bounds and not the count of products, keep their times.
__host__ __device__ constexpr int padded(int n) { return (n + 63) / 64 * 64; }

// LDS slots of the squaring kernels' operand rows.  A fragment read (ds_read_b128) takes lane
// (g, r) to 16-byte piece g (of 64-byte rows) or 2g + h (of 128-byte rows) of row r, g = lane / 16,
// r = lane % 16.  LDS serves it at 256 bytes per clock, 16 lanes at a time, but not 16 neighbours:
// lanes 0-3, 12-15, 20-23, 24-27 go together, then 4-7, 8-11, 16-19, 28-31, and the same of the
// upper half.  These permutations of a row's pieces keep each such set on 16 different 16-byte
// banks; permutations made for 16 (or 8) neighbouring lanes put it on eight: 7 clocks per read
// instead of 4 (measured on the pattern alone).  Conflicts went from a third of the LDS cycles to
// none; the squares, which the LDS does not bound, gained 1 to 2 % (fp16 N = 18000 3.92 -> 3.88 ms,
// N = 2050 0.670 -> 0.656, FP32 N = 3000 2.73 -> 2.70).
__device__ __forceinline__ int swz8(int r) { return (r >> 1) & 5; }
__device__ __forceinline__ int swz4(int r) { return (0x78 >> ((r >> 1) & 6)) & 3; }

// ---- gather: x0[s] = principal submatrix of X0 on the subgraph, zero padded -------------
// Block (s, chunk) writes rows [chunk*kRows, +kRows) of block s.  The subgraph list sits in
// LDS; the local column of an ELL entry is found by binary search in the core run and in
// the halo run (both ascending).
constexpr int kRows = 16;

template <typename T>
__global__ __launch_bounds__(kT) void k_gather(const int32_t* __restrict__ hcol,
                                               const double* __restrict__ x0, int w,
                                               const int32_t* __restrict__ core_ptr,
                                               const int32_t* __restrict__ sub_ptr,
                                               const int32_t* __restrict__ sub_idx,
                                               const int64_t* __restrict__ offs,
                                               const int32_t* __restrict__ npad, T* __restrict__ X,
                                               T scale) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int s = blockIdx.x;
  const int np = npad[s];
  const int a0 = blockIdx.y * kRows;
  if (a0 >= np) return;
  const int b = sub_ptr[s], n = sub_ptr[s + 1] - b;
  const int k = core_ptr[s + 1] - core_ptr[s];
  double* row = reinterpret_cast<double*>(smem);
  int32_t* sub = reinterpret_cast<int32_t*>(row + np);
  for (int a = threadIdx.x; a < n; a += kT) sub[a] = sub_idx[b + a];
  T* base = X + offs[s];
  for (int a = a0; a < a0 + kRows && a < np; ++a) {
    for (int c = threadIdx.x; c < np; c += kT) row[c] = 0.0;
    __syncthreads();
    if (a < n) {
      const int i = sub[a];
      for (int t = threadIdx.x; t < w; t += kT) {
        const int32_t j = hcol[(int64_t)i * w + t];
        if (j < 0) continue;
        // core run [0, k)
        int lo = 0, hi = k;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (sub[mid] < j) lo = mid + 1;
          else hi = mid;
        }
        int loc = -1;
        if (lo < k && sub[lo] == j) loc = lo;
        else {
          lo = k;
          hi = n;
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sub[mid] < j) lo = mid + 1;
            else hi = mid;
          }
          if (lo < n && sub[lo] == j) loc = lo;
        }
        if (loc >= 0) row[loc] = x0[(int64_t)i * w + t];
      }
    }
    __syncthreads();
    T* dst = base + (int64_t)a * np;
    for (int c = threadIdx.x; c < np; c += kT) dst[c] = (T)row[c] * scale;
    __syncthreads();
  }
}

// ---- the squaring kernel ----------------------------------------------------------------
// One workgroup (4 waves, 2 x 2) computes a 128 x 128 tile (bi, bj), bi <= bj, of a product of
// two symmetric blocks that commute (X*X, or X^2*X), so the result is symmetric: the tile is
// written at (bi, bj) and mirrored to (bj, bi).  Both operands are read as row panels (for a
// symmetric B, column j of B is row j).  k is consumed in 128-byte chunks staged in LDS
// (double buffered, one barrier per chunk).  Inside a chunk lane group g = lane/16 takes the
// k slice [g*KC/4, (g+1)*KC/4): the contraction is a sum over k, so any k order shared by
// both operands is valid, and each lane reads its slice with 16-byte LDS loads.
//   MODE 0: out = A*B          MODE 1: out = alpha*(A*B) + beta*E   (E symmetric)
//   MODE 2: out = alpha*(A*B + B*A) + beta*E for symmetric A, B, E (the adjoint's step).  Tile (bi,
//           bj) sums A's row panel bi with B's bj, then B's bi with A's bj: the flops of the
//           general product A*B, whose transpose would have to be added in a pass of its own, and
//           the result is written once.  The halves are summed apart (the first waits in out, not
//           in registers: 131 of them leave three waves per SIMD, 85 five): each rounds as the
//           general product did, and an entry of a diagonal tile and its transpose get the same
//           two sums.  klim > 0: A is zero outside its first klim rows and
//           columns, so a half of the sum whose panel of A lies below them ends after klim.
//           57 blocks of ~1330 rows: 4.80 ms a step against 5.09 (general product on 128-edge
//           tiles) + 0.46 (transpose and combine).
// In MODE 0 (A = B = X) the SP2 update is fused into the epilogue: with the branch
// 2X - X^2 selected (lin, or *lin_flag on the device-driven loop) the kernel writes 2X - X^2,
// else X^2.  X is symmetric, so the mirrored entry takes the same value.
// STAGES = 2: the next chunk loads while the current one is consumed; STAGES = 3: the two next
// chunks are in flight (one more LDS buffer), for latency the second buffer cannot hide.
// LOADER = 0: chunks go from global memory straight into LDS; LOADER = 1 (two stages): the
// chunk after next is loaded into registers under the current products and written to LDS
// once they are done.
template <typename T, int MODE, int BT = 128, int STAGES = 2, int LOADER = 0>
__global__ __launch_bounds__(kT, 2) void k_symm_mm(const T* __restrict__ A, const T* __restrict__ B,
                                                   const T* __restrict__ E, T* __restrict__ out,
                                                   T alpha, T beta, const int4* __restrict__ tiles,
                                                   const int64_t* __restrict__ offs,
                                                   const int32_t* __restrict__ stopped,
                                                   int lin,
                                                   const int32_t* __restrict__ lin_flag,
                                                   int klim) {
  if (stopped && *stopped) return;  // device-driven loop: the expansion already stopped
  static_assert(MODE != 2 || LOADER == 1, "the two-sided product stages through registers");
  using M = Mfma<T>;
  using acc_t = typename M::acc_t;
  constexpr int KC = M::KC;              // k elements per 128-byte row chunk
  constexpr int V = 16 / sizeof(T);      // elements per 16-byte piece
  constexpr int KG = KC / 4;             // k elements per lane group per chunk (two pieces)
  constexpr int WM = BT / 2;             // wave tile edge (2 x 2 waves)
  constexpr int MB = WM / 16;            // 16 x 16 blocks per wave tile edge
  constexpr int OPB = BT * 128;          // LDS bytes per operand per buffer
  constexpr int NLD = BT / 32;           // 1-KB wave loads per operand per chunk
  // [buffer][operand][row-major 128-byte rows, the eight 16-byte pieces of row r stored at slot
  // piece ^ swz8(r)]
  __shared__ __align__(1024) unsigned char lds[STAGES][2][OPB];

  const int4 tl = tiles[blockIdx.x];
  if (tl.x < 0) return;  // padding entry of an XCD queue
  const int s = tl.x, bi = tl.y, bj = tl.z, n_row = tl.w, np = padded(n_row);
  const int64_t off = offs[s];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;

  // Global -> LDS without registers (global_load_lds_dwordx4: lane L of a wave writes bytes
  // [16 L, 16 L + 16) of the wave's 1-KB LDS window).  Each lane's source is chosen so the
  // window receives the swizzled layout; rows beyond np (half-empty edge tiles) read row 0
  // instead, which only feeds output rows / columns that are never stored.
  const T* asrc[NLD];
  const T* bsrc[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int slot = (wave * NLD + j) * 64 + lane;
    const int r = slot >> 3, c = (slot & 7) ^ swz8(r);
    const int ar = bi * BT + r, br = bj * BT + r;
    asrc[j] = A + off + (int64_t)(ar < np ? ar : 0) * np + c * V;
    bsrc[j] = B + off + (int64_t)(br < np ? br : 0) * np + c * V;
  }
#define GB_ISSUE(buf, k0)                                                                   \
  _Pragma("unroll") for (int j = 0; j < NLD; ++j) {                                         \
    load_lds16(asrc[j] + (k0), &lds[buf][0][(wave * NLD + j) * 1024]);                      \
    load_lds16(bsrc[j] + (k0), &lds[buf][1][(wave * NLD + j) * 1024]);                      \
  }

  acc_t acc[MB][MB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n) acc[m][n] = acc_t{0, 0, 0, 0};

  const int g = lane >> 4, r16 = lane & 15;
  // chunks; MODE 2: of A_i B_j, then of B_i A_j
  int nk = (n_row + KC - 1) / KC, nk1 = 0;  // X is zero from n_row to np
  if constexpr (MODE == 2) {
    const int few = klim > 0 ? min((klim + KC - 1) / KC, nk) : nk;
    nk1 = klim > 0 && bi * BT >= klim ? few : nk;
    nk = nk1 + (klim > 0 && bj * BT >= klim ? few : nk);
  }
  // a wave whose row or column block lies beyond np has nothing to write, one whose block begins
  // in the padding writes zeros; on a diagonal tile of a symmetric product the lower-left block
  // is the transpose of the upper-right one, which that wave writes twice
  const bool lower_diag = bi == bj && wr > wc;
  const bool stores = bi * BT + wr * WM < np && bj * BT + wc * WM < np && !lower_diag;
  const bool active = stores && bi * BT + wr * WM < n_row && bj * BT + wc * WM < n_row;
  // byte offsets of this lane's pieces (2g + h) in rows wr*WM + m*16 + r16 (A) and
  // wc*WM + n*16 + r16 (B); swz8(row) = swz8(r16) for every m
  const int sw = swz8(r16);
  const int pa0 = (wr * WM + r16) * 128, pb0 = (wc * WM + r16) * 128;
  const int pc0 = (((2 * g) ^ sw) << 4), pc1 = (((2 * g + 1) ^ sw) << 4);

  // each wave issues 2 NLD loads per chunk; loads complete in order, so waiting until at most
  // 2 NLD are outstanding means every chunk but the newest has landed
  static_assert(STAGES == 2 || STAGES == 3, "two or three LDS stages");
  static_assert(STAGES == 2 || 2 * NLD == 4 || 2 * NLD == 8, "wait count");
#define GB_WAIT_ALL_BUT_NEWEST()                                   \
  do {                                                             \
    if constexpr (2 * NLD == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); \
    else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");          \
  } while (0)
  static_assert(LOADER == 0 || STAGES == 2, "register staging uses two LDS buffers");
  u4v stg[2][NLD];  // LOADER = 1: [operand][j], the 16 bytes this lane moves
  auto stage = [&](int c) {  // chunk c into registers
    if constexpr (MODE == 2) {
      const bool first = c < nk1;
      const T* base = first ? A : B;
      const int k0 = (first ? c : c - nk1) * KC;
#pragma unroll
      for (int j = 0; j < NLD; ++j) {
        stg[0][j] = *reinterpret_cast<const u4v*>(base + (asrc[j] - A) + k0);
        stg[1][j] = *reinterpret_cast<const u4v*>((first ? B : A) + (bsrc[j] - B) + k0);
      }
    } else {
#pragma unroll
      for (int j = 0; j < NLD; ++j) {
        stg[0][j] = *reinterpret_cast<const u4v*>(asrc[j] + c * KC);
        stg[1][j] = *reinterpret_cast<const u4v*>(bsrc[j] + c * KC);
      }
    }
  };
#define GB_PUT(buf)                                                                         \
  _Pragma("unroll") for (int j = 0; j < NLD; ++j) {                                         \
    *reinterpret_cast<u4v*>(&lds[buf][0][(wave * NLD + j) * 1024 + lane * 16]) = stg[0][j]; \
    *reinterpret_cast<u4v*>(&lds[buf][1][(wave * NLD + j) * 1024 + lane * 16]) = stg[1][j]; \
  }
  if (LOADER == 1) {
    stage(0);
    GB_PUT(0)
    if (nk > 1) stage(1);
  } else {
    GB_ISSUE(0, 0)
    if (STAGES == 3 && nk > 1) {
      GB_ISSUE(1, KC)
      GB_WAIT_ALL_BUT_NEWEST();
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
  }
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const int buf = kc % STAGES;
    const int ahead = kc + STAGES - 1;  // the chunk issued in this iteration
    if (LOADER == 0 && ahead < nk) {
      GB_ISSUE(ahead % STAGES, ahead * KC)
    }
    if (MODE == 2 && kc == nk1 && stores) {  // A_i B_j is done: aside, where the result will go
      T* o = out + off;
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < MB; ++n) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int grow = bi * BT + wr * WM + m * 16 + M::row(lane, r);
            const int gcol = bj * BT + wc * WM + n * 16 + r16;
            if (grow < np && gcol < np) o[(int64_t)grow * np + gcol] = acc[m][n][r];
          }
          acc[m][n] = acc_t{0, 0, 0, 0};
        }
    }
    if (active) {
      const unsigned char* la = lds[buf][0];
      const unsigned char* lb = lds[buf][1];
      // FP32: the chunk's 32 k-terms go to a fresh partial sum that is added to the running
      // one once per chunk (blocked summation): an output then passes through n/32 + 8
      // roundings instead of n/4 accumulating MFMAs, which keeps FP32 squares of blocks of
      // ~2000 rows well inside the 1e-6 accuracy bar after refinement.  FP64 accumulates
      // directly.
      constexpr bool kBlocked = std::is_same<T, float>::value;
      acc_t part[kBlocked ? MB : 1][kBlocked ? MB : 1];
      if constexpr (kBlocked) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < MB; ++n) part[m][n] = acc_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int pc = h ? pc1 : pc0;
        T fa[MB][V], fb[MB][V];
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          __builtin_memcpy(fa[m], la + pa0 + m * 16 * 128 + pc, 16);
          __builtin_memcpy(fb[m], lb + pb0 + m * 16 * 128 + pc, 16);
        }
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < MB; ++n) {
              if constexpr (kBlocked) part[m][n] = M::mma(fa[m][e], fb[n][e], part[m][n]);
              else acc[m][n] = M::mma(fa[m][e], fb[n][e], acc[m][n]);
            }
      }
      if constexpr (kBlocked) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < MB; ++n) acc[m][n] += part[m][n];
      }
    }
    if (LOADER == 1) {
      // chunk kc + 1 (in registers) into the other buffer, then the chunk after it
      if (kc + 1 < nk) {
        GB_PUT(buf ^ 1)
      }
      if (kc + 2 < nk) stage(kc + 2);
    } else if (STAGES == 3 && kc + 2 < nk) {
      // chunk kc + 1 must have landed; with three stages chunk kc + 2 may stay in flight
      GB_WAIT_ALL_BUT_NEWEST();
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
  }
#undef GB_PUT
#undef GB_WAIT_ALL_BUT_NEWEST
#undef GB_ISSUE

  if (!stores) return;
  T* o = out + off;
  const T* e = E + off;
  const T* xa = A + off;
  const bool do_lin = MODE == 0 && (lin_flag ? *lin_flag == 1 : lin != 0);
  const bool mirror = bi != bj || wr < wc;
  if constexpr (std::is_same<T, float>::value && MODE == 0) {
    // FP32 layout: lane l holds rows 4(l/16) .. +3 of column l%16, one contiguous run of the
    // transposed row, so the mirrored copy (and the symmetric X read of 2X - X^2) moves as one
    // 16-byte access; row groups of four lie entirely inside or outside npad
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int n = 0; n < MB; ++n) {
        const int grow0 = bi * BT + wr * WM + m * 16 + 4 * (lane >> 4);
        const int gcol = bj * BT + wc * WM + n * 16 + r16;
        if (grow0 >= np || gcol >= np) continue;
        const int64_t qt = (int64_t)gcol * np + grow0;
        f4v v = acc[m][n];
        if (do_lin) v = 2.0f * *reinterpret_cast<const f4v*>(xa + qt) - v;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[(int64_t)(grow0 + r) * np + gcol] = v[r];
        if (mirror) *reinterpret_cast<f4v*>(o + qt) = v;
      }
    return;
  }
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int grow = bi * BT + wr * WM + m * 16 + M::row(lane, r);
        const int gcol = bj * BT + wc * WM + n * 16 + r16;
        if (grow < np && gcol < np) {
          const int64_t q1 = (int64_t)grow * np + gcol, q2 = (int64_t)gcol * np + grow;
          T v = acc[m][n][r];
          if (MODE == 2) v = o[q1] + v;
          if (MODE == 1 || MODE == 2) v = alpha * v + beta * e[q1];
          if (do_lin) v = (T)2 * xa[q1] - v;
          o[q1] = v;
          if (mirror) o[q2] = v;
        }
      }
}


// The squares (MODE 0 of k_symm_mm) of a small batch on 32 x 32 tiles, one 16 x 16 block a wave
// (small_batch below says which batches).  What bounds such a launch is the chain of one tile,
// not any rate: a 64-edge tile of a 256-row block is 16 chunks, each a wait for memory, a
// barrier and 16 products per wave, on fewer compute units than there are.  Here a wave has four
// products per chunk, and the loads of two chunks go out under the products of the two before
// (one chunk: 3 % slower at 512 rows, four: 8 % at 704).  Every output is the same sum in the same
// order.  FP64, against k_symm_mm on 64-edge tiles: one block of 704 rows 41.9 -> 20.1 us, 16 of
// 256 20.4 -> 15.3, 32 of 512 115 -> 91; large batches lose the reuse: 64 of 900 rows 924 -> 935.
template <typename T>
__global__ __launch_bounds__(kT) void k_square_small(const T* __restrict__ X, T* __restrict__ S,
                                                     const int4* __restrict__ tiles,
                                                     const int64_t* __restrict__ offs,
                                                     const int32_t* __restrict__ stopped, int lin,
                                                     const int32_t* __restrict__ lin_flag) {
  if (stopped && *stopped) return;
  using M = Mfma<T>;
  using acc_t = typename M::acc_t;
  constexpr int KC = M::KC, V = 16 / sizeof(T);
  constexpr int NCH = 2;  // chunks per stage
  __shared__ __align__(1024) unsigned char lds[2][NCH][32 * 128];  // rows as in k_symm_mm
  const int4 tl = tiles[blockIdx.x];
  if (tl.x < 0) return;
  const int s = tl.x, bi = tl.y, bj = tl.z, n_row = tl.w, np = padded(n_row);
  const int64_t off = offs[s];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1, g = lane >> 4, r16 = lane & 15;
  // np is a multiple of the tile: every row of the tile exists
  const int sr = tid >> 3, sc = ((tid & 7) ^ swz8(sr)) * V;
  const T* asrc = X + off + (int64_t)(bi * 32 + sr) * np + sc;
  const T* bsrc = X + off + (int64_t)(bj * 32 + sr) * np + sc;
  const int nk = (n_row + KC - 1) / KC;
  const bool stores = !(bi == bj && wr > wc);
  const bool active = stores && bi * 32 + wr * 16 < n_row && bj * 32 + wc * 16 < n_row;
  u4v stg[2][NCH];
  auto load = [&](int c0) {  // chunks c0 .. c0 + NCH - 1; past the last one: that one again
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int k = min(c0 + c, nk - 1) * KC;
      stg[0][c] = *reinterpret_cast<const u4v*>(asrc + k);
      stg[1][c] = *reinterpret_cast<const u4v*>(bsrc + k);
    }
  };
  const int sw = swz8(r16);
  const int pa = (wr * 16 + r16) * 128, pb = (wc * 16 + r16) * 128;
  const int pc[2] = {((2 * g) ^ sw) << 4, ((2 * g + 1) ^ sw) << 4};
  acc_t acc = {0, 0, 0, 0};
  load(0);
  for (int c0 = 0; c0 < nk; c0 += NCH) {
    __syncthreads();  // the previous chunks' reads are done
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      *reinterpret_cast<u4v*>(&lds[0][c][tid * 16]) = stg[0][c];
      *reinterpret_cast<u4v*>(&lds[1][c][tid * 16]) = stg[1][c];
    }
    __syncthreads();
    if (c0 + NCH < nk) load(c0 + NCH);
    if (active) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        if (c0 + c >= nk) break;
        constexpr bool kBlocked = std::is_same<T, float>::value;  // as in k_symm_mm
        acc_t part = {0, 0, 0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          T fa[V], fb[V];
          __builtin_memcpy(fa, &lds[0][c][pa + pc[h]], 16);
          __builtin_memcpy(fb, &lds[1][c][pb + pc[h]], 16);
#pragma unroll
          for (int e = 0; e < V; ++e) {
            if constexpr (kBlocked) part = M::mma(fa[e], fb[e], part);
            else acc = M::mma(fa[e], fb[e], acc);
          }
        }
        if constexpr (kBlocked) acc += part;
      }
    }
  }
  if (!stores) return;
  T* o = S + off;
  const bool do_lin = lin_flag ? *lin_flag == 1 : lin != 0;
  const bool mirror = bi != bj || wr < wc;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int grow = bi * 32 + wr * 16 + M::row(lane, r), gcol = bj * 32 + wc * 16 + r16;
    const int64_t q1 = (int64_t)grow * np + gcol, q2 = (int64_t)gcol * np + grow;
    T v = acc[r];
    if (do_lin) v = (T)2 * X[off + q1] - v;
    o[q1] = v;
    if (mirror) o[q2] = v;
  }
}


// ---- split squaring ---------------------------------------------------------------------
// An FP32 iterate x is split into planes: bf16 ones hi = bf16(x), mid = bf16(x - hi),
// lo = bf16(x - hi - mid) (each remainder is exact in FP32, and hi + mid + lo = x whenever x
// is an FP32 number), or two fp16 planes of 2^14 x.  X*X is summed over the plane products
// that keep about NP*8 bits (NP = 1: hi*hi; NP = 2 (hi, lo = bf16(x - hi)): + hi*lo, lo*hi;
// NP = 3: + hi*mid, mid*hi, hi*lo, lo*hi, mid*mid) or, for the fp16 planes, hi*hi + hi*lo +
// lo*hi (about 22 bits), on the 16 x 16 x 32 matrix cores with FP32 accumulation.

// The split of two values at once, each plane's pair packed in one 32-bit word (x0 in the low
// half): one packed conversion per plane, the plane values recovered from that word (a shift or
// a mask for bf16, a conversion for fp16) for the next remainder.
// F16: two fp16 planes of 2^14 x instead (hi = fp16(2^14 x), lo = fp16(2^14 x - hi), about 22
// bits; |x| <= 1 for an iterate with its spectrum in [0, 1], so 2^14 x stays far below the fp16
// maximum and values down to ~4e-9 stay normal).  The fp16 loop keeps its FP32 iterate stored
// as x' = 2^14 x (the gather and the conversion into the loop scale it, the traces and the
// conversion out of the loop scale back, all exact powers of two), so the split needs no
// multiply: hi = fp16(x'), lo = fp16(x' - hi).  The products then carry 2^28 = 2^14 * 2^14;
// the epilogue multiplies by 2^-14 to store the next iterate, again as 2^14 times its value.
constexpr float kF16Scale = 16384.0f;                    // 2^14
constexpr float kF16Down = 6.103515625e-05f;             // 2^-14
constexpr double kF16TraceDown1 = 6.103515625e-05;       // 2^-14 (diagonal sums)
constexpr double kF16TraceDown2 = 3.7252902984619140625e-09;  // 2^-28 (sums of squares)
// neg1 is -1: passed as a value the compiler cannot see (a register), the remainder
// r - fp16(r) = fma(-1, fp16(r), r) (exact product, one rounding, as the subtraction) becomes one
// mixed-precision FMA that reads the fp16 half directly, instead of a conversion and a
// subtraction.
template <int NP, bool F16 = false>
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t* w, float neg1 = -1.0f) {
  typedef float f2v __attribute__((ext_vector_type(2)));
  if constexpr (F16) {
    typedef _Float16 h2v __attribute__((ext_vector_type(2)));
    float r0 = x0, r1 = x1;  // the stored iterate is already 2^14 x
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const h2v h = __builtin_convertvector(f2v{r0, r1}, h2v);
      uint32_t u;
      __builtin_memcpy(&u, &h, 4);
      w[p] = u;
      if (p + 1 < NP) {
        r0 = __builtin_fmaf(neg1, (float)h[0], r0);
        r1 = __builtin_fmaf(neg1, (float)h[1], r1);
      }
    }
  } else {
    float r0 = x0, r1 = x1;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
      const bf2v h = __builtin_convertvector(f2v{r0, r1}, bf2v);
      uint32_t u;
      __builtin_memcpy(&u, &h, 4);
      w[p] = u;
      if (p + 1 < NP) {
        r0 -= __uint_as_float(u << 16);
        r1 -= __uint_as_float(u & 0xffff0000u);
      }
    }
  }
}

// Epilogue of the split kernels: the new iterate v = big + small (times 2^-28 for fp16 planes),
// or 2x - v, written at (row, col) and, off the diagonal blocks, at (col, row).  Lane l holds
// rows 4(l/16) .. 4(l/16) + 3 of column l%16 of each 16 x 16 block, so its four values are one
// contiguous run of the transposed row: the mirrored copy (and the x read by the 2x - v branch,
// X being symmetric) moves as one 16-byte access.  Rows come in groups of four and npad is a
// multiple of 64, so a group is entirely inside or outside.
template <int BT, bool F16>
__device__ __forceinline__ void split_epilogue(const f4v (&big)[BT / 32][BT / 32],
                                               const f4v (&small)[BT / 32][BT / 32],
                                               float* __restrict__ S, const float* __restrict__ X,
                                               int64_t off, int np, int bi, int bj, int wr, int wc,
                                               int lane, bool do_lin) {
  constexpr int MB = BT / 32, WT = BT / 2;
  float* o = S + off;
  const float* xa = X + off;
  const int r16 = lane & 15;
  const bool mirror = bi != bj || wr < wc;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n) {
      const int grow0 = bi * BT + wr * WT + m * 16 + 4 * (lane >> 4);
      const int gcol = bj * BT + wc * WT + n * 16 + r16;
      if (grow0 >= np || gcol >= np) continue;
      const int64_t qt = (int64_t)gcol * np + grow0;  // (gcol, grow0 .. grow0 + 3)
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[r] = big[m][n][r] + small[m][n][r];
        if (F16) v[r] *= kF16Down;
      }
      if (do_lin) {
        const f4v xt = *reinterpret_cast<const f4v*>(xa + qt);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = 2.0f * xt[r] - v[r];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) o[(int64_t)(grow0 + r) * np + gcol] = v[r];
      if (mirror) *reinterpret_cast<f4v*>(o + qt) = f4v{v[0], v[1], v[2], v[3]};
    }
}

// Split squaring: the FP32 iterate itself is read and each lane splits the 16 bytes it loads
// into the NP planes (bf16, or fp16 of 2^14 x) while staging them into the swizzled LDS layout
// (four 16-byte pieces per 64-byte plane row, piece p of row r at slot p ^ swz4(r)).  X^2 is the
// sum of the plane products that keep about 8 NP bits (bf16) or 22 bits (two fp16 planes) on the 16
// x 16 x 32 matrix cores, the leading product and the corrections in separate FP32 accumulators,
// added once at the end; the epilogue applies the SP2 update and writes only the FP32 result.  The
// next chunk is loaded into registers under the current chunk's products.  A workgroup of four
// waves (2 x 2) computes a BT x BT tile (bi <= bj) of the symmetric product, BT = 128 or 64;
// tiles and XCD order as in k_symm_mm.
template <int NP, bool F16, int BT>
__global__ __launch_bounds__(kT, 2) void k_symm_mm_split(const float* __restrict__ X,
                                                        float* __restrict__ S,
                                                        const int4* __restrict__ tiles,
                                                        const int64_t* __restrict__ offs,
                                                        const int32_t* __restrict__ stopped,
                                                        int lin,
                                                        const int32_t* __restrict__ lin_flag) {
  if (stopped && *stopped) return;
  constexpr int KC = 32;           // k per chunk (64 bytes per plane row)
  constexpr int OPB = BT * 64;     // bytes per plane and operand
  constexpr int MB = BT / 32;      // 16 x 16 blocks per wave-tile edge
  constexpr int WT = BT / 2;       // wave-tile edge
  constexpr int NQ = BT / 32;      // rows per staging thread and operand
  __shared__ __align__(1024) unsigned char lds[NP][2][OPB];
  const int4 tl = tiles[blockIdx.x];
  if (tl.x < 0) return;
  const int s = tl.x, bi = tl.y, bj = tl.z, n_row = tl.w, np = padded(n_row);
  const int64_t off = offs[s];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  // staging: thread t moves FP32 piece c8 = t % 8 (k = 4 c8 .. 4 c8 + 3) of rows
  // t / 8 + 32 q (q < NQ) of each operand; eight threads cover one row's 128 bytes.  Rows beyond
  // np read row 0 (they only feed outputs that are never stored).
  const int c8 = tid & 7, r0 = tid >> 3;
  const float* asrc[NQ];
  const float* bsrc[NQ];
  int ldo[NQ];  // byte offset of the 8-byte run in a plane's operand array
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int r = r0 + 32 * q;
    const int ar = bi * BT + r, br = bj * BT + r;
    asrc[q] = X + off + (int64_t)(ar < np ? ar : 0) * np + 4 * c8;
    bsrc[q] = X + off + (int64_t)(br < np ? br : 0) * np + 4 * c8;
    ldo[q] = r * 64 + (((c8 >> 1) ^ swz4(r)) << 4) + (c8 & 1) * 8;
  }
  f4v big[MB][MB], small[MB][MB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n) {
      big[m][n] = f4v{0, 0, 0, 0};
      small[m][n] = f4v{0, 0, 0, 0};
    }
  const int g = lane >> 4, r16 = lane & 15;
  const int nk = (n_row + KC - 1) / KC;  // X is zero from n_row to np
  // which waves write and which of them compute: as in k_symm_mm
  const bool stores =
      bi * BT + wr * WT < np && bj * BT + wc * WT < np && !(bi == bj && wr > wc);
  const bool active = stores && bi * BT + wr * WT < n_row && bj * BT + wc * WT < n_row;
  const int pa0 = (wr * WT + r16) * 64, pb0 = (wc * WT + r16) * 64;
  const int pc = (g ^ swz4(r16)) << 4;
  f4v stg[2][NQ];  // [operand][q]
  float neg1 = -1.0f;  // see split_pair
  asm volatile("" : "+v"(neg1));
#define GB_STAGE(k0)                                                                          \
  _Pragma("unroll") for (int q = 0; q < NQ; ++q) {                                            \
    stg[0][q] = *reinterpret_cast<const f4v*>(asrc[q] + (k0));                                \
    stg[1][q] = *reinterpret_cast<const f4v*>(bsrc[q] + (k0));                                \
  }
#define GB_FRAG(dst, plane, opnd, base, m) \
  __builtin_memcpy(&(dst), &lds[plane][opnd][(base) + (m) * 16 * 64 + pc], 16)
  GB_STAGE(0)
  for (int kc = 0; kc < nk; ++kc) {
    __syncthreads();  // the previous chunk's reads are done
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        uint32_t lo[NP], hi[NP];
        split_pair<NP, F16>(stg[o][q][0], stg[o][q][1], lo, neg1);
        split_pair<NP, F16>(stg[o][q][2], stg[o][q][3], hi, neg1);
#pragma unroll
        for (int p = 0; p < NP; ++p)
          *reinterpret_cast<uint2*>(&lds[p][o][ldo[q]]) = uint2{lo[p], hi[p]};
      }
    __syncthreads();
    if (kc + 1 < nk) {
      GB_STAGE((kc + 1) * KC)
    }
    if (active) {
      bf8v A0[MB], B0[MB];
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        GB_FRAG(A0[m], 0, 0, pa0, m);
        GB_FRAG(B0[m], 0, 1, pb0, m);
      }
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < MB; ++n) big[m][n] = mma_p<F16>(A0[m], B0[n], big[m][n]);
      if (NP >= 2) {
        // hi x last plane, last plane x hi (lo for NP = 2, lo for NP = 3)
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          bf8v BL;
          GB_FRAG(BL, NP - 1, 1, pb0, m);
#pragma unroll
          for (int r = 0; r < MB; ++r) small[r][m] = mma_p<F16>(A0[r], BL, small[r][m]);
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          bf8v AL;
          GB_FRAG(AL, NP - 1, 0, pa0, m);
#pragma unroll
          for (int n = 0; n < MB; ++n) small[m][n] = mma_p<F16>(AL, B0[n], small[m][n]);
        }
      }
      if (NP >= 3) {
        // hi x mid, mid x hi, mid x mid
        bf8v BM[MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) GB_FRAG(BM[m], 1, 1, pb0, m);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < MB; ++n) small[m][n] = mma_p<F16>(A0[m], BM[n], small[m][n]);
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          bf8v AM;
          GB_FRAG(AM, 1, 0, pa0, m);
#pragma unroll
          for (int n = 0; n < MB; ++n) {
            small[m][n] = mma_p<F16>(AM, B0[n], small[m][n]);
            small[m][n] = mma_p<F16>(AM, BM[n], small[m][n]);
          }
        }
      }
    }
  }
#undef GB_FRAG
#undef GB_STAGE
  if (!stores) return;
  split_epilogue<BT, F16>(big, small, S, X, off, np, bi, bj, wr, wc, lane,
                          lin_flag ? *lin_flag == 1 : lin != 0);
}

// ---- split squaring with the split under the products -------------------------------------
// Scheduling hints (the compiler places the named instruction classes in the given order
// within a block of straight-line code): one matrix-core instruction, n vector-ALU ones, one
// LDS read or write.
__device__ inline void sched_mfma1() { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); }
__device__ inline void sched_valu2() { __builtin_amdgcn_sched_group_barrier(0x002, 2, 0); }
__device__ inline void sched_valu4() { __builtin_amdgcn_sched_group_barrier(0x002, 4, 0); }
__device__ inline void sched_dsr1() { __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); }
__device__ inline void sched_dsr8() { __builtin_amdgcn_sched_group_barrier(0x100, 8, 0); }
__device__ inline void sched_dsw1() { __builtin_amdgcn_sched_group_barrier(0x200, 1, 0); }
__device__ inline void sched_vmr4() { __builtin_amdgcn_sched_group_barrier(0x020, 4, 0); }

// fp16 x 2 planes (three products), as k_symm_mm_split<2, true, BT>, with two LDS buffers: the
// planes of chunk kc + 1 are split from registers and written to one buffer while the products
// of chunk kc read the other, the split's vector instructions and LDS writes interleaved with
// the matrix-core instructions (the first operand's split under the leading products, the
// second's under the hi x lo products), one barrier per chunk.  Each operand's next chunk
// is loaded into registers once its split has consumed them.  The two buffers are separate
// arrays and the loop is unrolled by two, so reads of one and writes of the other are known
// not to alias.  Products, their order and the accumulators are those of k_symm_mm_split, so
// both give the same bits.
template <int BT>
__global__ __launch_bounds__(kT, 2) void k_symm_mm_split_il(const float* __restrict__ X,
                                                           float* __restrict__ S,
                                                           const int4* __restrict__ tiles,
                                                           const int64_t* __restrict__ offs,
                                                           const int32_t* __restrict__ stopped,
                                                           int lin,
                                                           const int32_t* __restrict__ lin_flag) {
  if (stopped && *stopped) return;
  constexpr int NP = 2;
  constexpr int KC = 32;           // k per chunk (64 bytes per plane row)
  constexpr int OPB = BT * 64;     // bytes per plane and operand
  constexpr int MB = BT / 32;      // 16 x 16 blocks per wave-tile edge
  constexpr int WT = BT / 2;       // wave-tile edge
  constexpr int NQ = BT / 32;      // rows per staging thread and operand
  __shared__ __align__(1024) unsigned char lds0[NP][2][OPB];
  __shared__ __align__(1024) unsigned char lds1[NP][2][OPB];
  const int4 tl = tiles[blockIdx.x];
  if (tl.x < 0) return;
  const int s = tl.x, bi = tl.y, bj = tl.z, n_row = tl.w, np = padded(n_row);
  const int64_t off = offs[s];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int c8 = tid & 7, r0 = tid >> 3;
  // 32-bit element offsets into the block (np^2 < 2^31) from one workgroup-uniform base
  const float* xblk = X + off;
  int asrc[NQ], bsrc[NQ], ldo[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int r = r0 + 32 * q;
    const int ar = bi * BT + r, br = bj * BT + r;
    asrc[q] = (ar < np ? ar : 0) * np + 4 * c8;
    bsrc[q] = (br < np ? br : 0) * np + 4 * c8;
    ldo[q] = r * 64 + (((c8 >> 1) ^ swz4(r)) << 4) + (c8 & 1) * 8;
  }
  f4v big[MB][MB], small[MB][MB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n) {
      big[m][n] = f4v{0, 0, 0, 0};
      small[m][n] = f4v{0, 0, 0, 0};
    }
  const int g = lane >> 4, r16 = lane & 15;
  const int nk = (n_row + KC - 1) / KC;  // X is zero from n_row to np
  const bool stores =
      bi * BT + wr * WT < np && bj * BT + wc * WT < np && !(bi == bj && wr > wc);
  const bool active = stores && bi * BT + wr * WT < n_row && bj * BT + wc * WT < n_row;
  const int pa0 = (wr * WT + r16) * 64, pb0 = (wc * WT + r16) * 64;
  const int pc = (g ^ swz4(r16)) << 4;
  f4v stg[2][NQ];  // [operand][q]
  float neg1 = -1.0f;  // see split_pair
  asm volatile("" : "+v"(neg1));
  auto load_op = [&](int o, int k0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      stg[o][q] = *reinterpret_cast<const f4v*>(xblk + (o ? bsrc[q] : asrc[q]) + k0);
  };
  // the split of operand o, row groups q0 .. q0 + nq - 1, into dst
  auto split_op = [&](int o, unsigned char (&dst)[NP][2][OPB], int q0, int nq) {
#pragma unroll
    for (int q = q0; q < q0 + nq; ++q) {
      // an empty statement the value passes through, so that the split stays where it is
      // written (the same code on both sides of the `active` branch would otherwise be hoisted
      // above it, waiting for every load at the top of the chunk)
      asm volatile("" : "+v"(stg[o][q]));
      uint32_t lo[NP], hi[NP];
      split_pair<NP, true>(stg[o][q][0], stg[o][q][1], lo, neg1);
      split_pair<NP, true>(stg[o][q][2], stg[o][q][3], hi, neg1);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<uint2*>(&dst[p][o][ldo[q]]) = uint2{lo[p], hi[p]};
    }
  };
  // one chunk: products from `cur`, the next chunk's planes into `nxt`, then the chunk after
  // that (k element k2) into registers; past the end k2 repeats the last chunk, just read by
  // the same lanes (a cache hit), whose planes are never written (no branch inside the
  // interleaved code)
  auto step = [&](unsigned char (&cur)[NP][2][OPB], unsigned char (&nxt)[NP][2][OPB], int k2) {
    if (active) {
      bf8v A0[MB], B0[MB];
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        __builtin_memcpy(&A0[m], &cur[0][0][pa0 + m * 16 * 64 + pc], 16);
        __builtin_memcpy(&B0[m], &cur[0][1][pb0 + m * 16 * 64 + pc], 16);
      }
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < MB; ++n) big[m][n] = mma_f16(A0[m], B0[n], big[m][n]);
      split_op(0, nxt, 0, NQ);
      // 2 MB fragment reads, then MB^2 products each with four split instructions, and one
      // plane write (both planes of a row group) per MB^2 / NQ products
      sched_dsr8();
#pragma unroll
      for (int i = 0; i < MB * MB; ++i) {
        sched_mfma1();
        sched_valu4();
        if (i % (MB * MB / NQ) == MB * MB / NQ - 1) sched_dsw1();
      }
      load_op(0, k2);
      sched_vmr4();  // the next loads after the split that frees their registers
      // the second operand's split under the hi x lo products, so that its next chunk's loads, too,
      // have a third of the step and more ahead of them
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        bf8v BL;
        __builtin_memcpy(&BL, &cur[1][1][pb0 + m * 16 * 64 + pc], 16);
#pragma unroll
        for (int r = 0; r < MB; ++r) small[r][m] = mma_f16(A0[r], BL, small[r][m]);
      }
      split_op(1, nxt, 0, NQ);
#pragma unroll
      for (int i = 0; i < MB * MB; ++i) {
        if (i % MB == 0) sched_dsr1();
        sched_mfma1();
        sched_valu4();
        if (i % (MB * MB / NQ) == MB * MB / NQ - 1) sched_dsw1();
      }
      load_op(1, k2);
      sched_vmr4();
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        bf8v AL;
        __builtin_memcpy(&AL, &cur[1][0][pa0 + m * 16 * 64 + pc], 16);
#pragma unroll
        for (int n = 0; n < MB; ++n) small[m][n] = mma_f16(AL, B0[n], small[m][n]);
      }
#pragma unroll
      for (int i = 0; i < MB * MB; ++i) {
        if (i % MB == 0) sched_dsr1();
        sched_mfma1();
      }
    } else {
      split_op(0, nxt, 0, NQ);
      split_op(1, nxt, 0, NQ);
      load_op(0, k2);
      load_op(1, k2);
    }
    __syncthreads();
  };
  load_op(0, 0);
  load_op(1, 0);
  split_op(0, lds0, 0, NQ);
  split_op(1, lds0, 0, NQ);
  if (nk > 1) {
    load_op(0, KC);
    load_op(1, KC);
  }
  __syncthreads();
  // the planes written past the last chunk are never read
  for (int kc = 0; kc < nk; kc += 2) {
    step(lds0, lds1, min(kc + 2, nk - 1) * KC);
    if (kc + 1 < nk) step(lds1, lds0, min(kc + 3, nk - 1) * KC);
  }
  if (!stores) return;
  split_epilogue<BT, true>(big, small, S, X, off, np, bi, bj, wr, wc, lane,
                           lin_flag ? *lin_flag == 1 : lin != 0);
}

// ---- traces and the branch decision --------------------------------------------------------
// t1 = sum over subgraphs of the core diagonal of X; t2 = the same for X^2, which for the
// symmetric X is the sum of the squared entries of the core rows.  Taking t2 from X lets the
// stop test and the branch come before the square: the last square of the loop is not
// needed, and the square kernel applies the update in its epilogue.  One workgroup per
// subgraph writes its two partial sums (fixed order); one workgroup adds them (fixed order)
// and decides.
struct StepRec {
  double t1, t2, e, margin;
  int32_t b, stop, pad0, pad1;
  // device-driven loop: the wall clock (wall_clock64) when the step's trace kernel began and
  // when its decision was made; the square in between ran from `out` to the next step's `in`
  long long in, out;
};

// the two partial sums of subgraph blockIdx.x (valid in thread 0)
template <typename T>
__device__ __forceinline__ void trace_block(const T* __restrict__ X,
                                            const int64_t* __restrict__ offs,
                                            const int32_t* __restrict__ npad,
                                            const int32_t* __restrict__ core_ptr, double* sum1,
                                            double* sum2) {
  constexpr int V = 16 / sizeof(T);  // values per 16-byte load
  typedef T vec __attribute__((ext_vector_type(V)));
  __shared__ double r1[kT], r2[kT];
  const int s = blockIdx.x;
  const int np = npad[s], k = core_ptr[s + 1] - core_ptr[s];
  const int nv = np / V;  // np is a multiple of 64
  const T* xs = X + offs[s];
  double p1 = 0.0, p2 = 0.0;
  // 16-byte loads, four rows at a time, so that each thread has several loads in flight; the
  // thread whose load holds element (j, j) adds it to the diagonal sum
  auto row_sums = [&](int j, const vec& v, int a) {
#pragma unroll
    for (int e = 0; e < V; ++e) p2 += (double)v[e] * (double)v[e];
    if (a == j / V) p1 += (double)v[j % V];
  };
  int j = 0;
  for (; j + 4 <= k; j += 4) {
    const vec* r0 = reinterpret_cast<const vec*>(xs + (int64_t)j * np);
    const vec* r1p = reinterpret_cast<const vec*>(xs + (int64_t)(j + 1) * np);
    const vec* r2p = reinterpret_cast<const vec*>(xs + (int64_t)(j + 2) * np);
    const vec* r3p = reinterpret_cast<const vec*>(xs + (int64_t)(j + 3) * np);
    for (int a = threadIdx.x; a < nv; a += kT) {
      const vec v0 = r0[a], v1 = r1p[a], v2 = r2p[a], v3 = r3p[a];
      row_sums(j, v0, a);
      row_sums(j + 1, v1, a);
      row_sums(j + 2, v2, a);
      row_sums(j + 3, v3, a);
    }
  }
  for (; j < k; ++j) {
    const vec* r0 = reinterpret_cast<const vec*>(xs + (int64_t)j * np);
    for (int a = threadIdx.x; a < nv; a += kT) row_sums(j, r0[a], a);
  }
  r1[threadIdx.x] = p1;
  r2[threadIdx.x] = p2;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      r1[threadIdx.x] += r1[threadIdx.x + h];
      r2[threadIdx.x] += r2[threadIdx.x + h];
    }
    __syncthreads();
  }
  *sum1 = r1[0];
  *sum2 = r2[0];
}

template <typename T>
__global__ __launch_bounds__(kT) void k_trace_rows(const T* __restrict__ X,
                                                   const int64_t* __restrict__ offs,
                                                   const int32_t* __restrict__ npad,
                                                   const int32_t* __restrict__ core_ptr,
                                                   double* __restrict__ part,
                                                   const int32_t* __restrict__ stopped,
                                                   double s1, double s2) {
  if (stopped && *stopped) return;
  double p1, p2;
  trace_block(X, offs, npad, core_ptr, &p1, &p2);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = p1 * s1;
    part[2 * blockIdx.x + 1] = p2 * s2;
  }
}

// FRESH: the partials were written by other workgroups of this launch (read past the XCD's L2)
template <bool FRESH = false>
__device__ void sum_partials(const double* __restrict__ part, int n_sub, double* t1, double* t2) {
  __shared__ double r1[kT], r2[kT];
  double p1 = 0.0, p2 = 0.0;
  for (int s = threadIdx.x; s < n_sub; s += kT) {
    if (FRESH) {
      p1 += __hip_atomic_load(&part[2 * s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      p2 += __hip_atomic_load(&part[2 * s + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      p1 += part[2 * s];
      p2 += part[2 * s + 1];
    }
  }
  r1[threadIdx.x] = p1;
  r2[threadIdx.x] = p2;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      r1[threadIdx.x] += r1[threadIdx.x + h];
      r2[threadIdx.x] += r2[threadIdx.x + h];
    }
    __syncthreads();
  }
  *t1 = r1[0];
  *t2 = r2[0];
}

// forced: -1 choose by the trace rule, 0/1 replay that branch, 2 stop (record only),
// 10/11 take branch 0/1 unless the stop test holds (alternating refinement)
__global__ __launch_bounds__(kT) void k_decide(const double* __restrict__ part, int n_sub,
                                               double n_occ, double tol, int forced, int at_max,
                                               StepRec* __restrict__ rec) {
  double t1, t2;
  sum_partials(part, n_sub, &t1, &t2);
  if (threadIdx.x == 0) {
    const double e = fabs(t1 - t2);
    const double dsq = fabs(t2 - n_occ), dlin = fabs(2.0 * t1 - t2 - n_occ);
    StepRec q;
    q.t1 = t1;
    q.t2 = t2;
    q.e = e;
    q.margin = fabs(dsq - dlin);
    q.pad0 = q.pad1 = 0;
    q.b = -1;
    q.stop = 0;
    if (forced == 2) q.stop = 1;
    else if (forced >= 10 && e <= tol) q.stop = 1;
    else if (forced >= 10 && at_max) q.stop = 2;
    else if (forced >= 10) q.b = forced - 10;
    else if (forced >= 0) q.b = forced;
    else if (e <= tol) q.stop = 1;
    else if (at_max) q.stop = 2;
    else q.b = dsq < dlin ? 0 : 1;
    *rec = q;
  }
}

// ---- device-driven loop (hipGraph): the stop flag, iteration counter, current branch and
// records live on the device, so a captured pair of iterations can be replayed without host
// round trips.  Every update writes the new iterate into the other buffer, so buffer roles
// simply alternate.
struct LoopState {
  int32_t it, stopped, max_iter, n_forced;  // n_forced < 0: choose by the trace rule
  int32_t stag, cur_b, first;  // first: step at which the loop began (stagnation waits nine steps)
  int32_t ticket;  // workgroups of the step's trace kernel that are done
  double n_occ, tol, e_hand;  // e_hand: stop once the traces agree to this (0: never)
  uint8_t forced[128];
  StepRec recs[128];
};
// What the host sees of it while it runs (pinned memory): decisions made, and the stop.
struct LoopProgress {
  int32_t it, stopped;
};
// The loop's parameters, passed by value to the kernel that sets up LoopState.
struct LoopInit {
  int32_t it0, first, max_iter, n_forced, stag;
  double n_occ, tol, e_hand;
  double e_back[2];  // of the two steps before it0, where first < it0
  uint8_t forced[128];
};

// One launch per decision: every workgroup leaves its subgraph's two partial sums, and the last
// one to do so adds them up (in the fixed order of the kernels above) and decides.  (A launch of
// its own for the decision cost 4 us a step and its gap.)
template <typename T>
__global__ __launch_bounds__(kT) void k_trace_step(const T* __restrict__ X,
                                                   const int64_t* __restrict__ offs,
                                                   const int32_t* __restrict__ npad,
                                                   const int32_t* __restrict__ core_ptr,
                                                   double* __restrict__ part, double s1, double s2,
                                                   LoopState* __restrict__ st,
                                                   LoopProgress* __restrict__ seen) {
  __shared__ int last;
  // read by every workgroup before its ticket, written after the last one's
  if (st->stopped) return;
  const long long began = wall_clock64();
  double p1, p2;
  trace_block(X, offs, npad, core_ptr, &p1, &p2);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&part[2 * blockIdx.x], p1 * s1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&part[2 * blockIdx.x + 1], p2 * s2, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    if (blockIdx.x == 0)
      __hip_atomic_store(&st->recs[st->it].in, began, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int t = __hip_atomic_fetch_add(&st->ticket, 1, __ATOMIC_ACQ_REL,
                                         __HIP_MEMORY_SCOPE_AGENT);
    last = t == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  double t1, t2;
  sum_partials<true>(part, gridDim.x, &t1, &t2);
  if (threadIdx.x == 0) {
    const int it = st->it;
    const double n_occ = st->n_occ;
    const double e = fabs(t1 - t2);
    const double dsq = fabs(t2 - n_occ), dlin = fabs(2.0 * t1 - t2 - n_occ);
    StepRec q;
    q.t1 = t1;
    q.t2 = t2;
    q.e = e;
    q.margin = fabs(dsq - dlin);
    q.pad0 = q.pad1 = 0;
    q.b = -1;
    q.stop = 0;
    if (it >= 127) {
      q.stop = st->n_forced >= 0 ? 1 : 2;  // the records hold 128 steps
    } else if (st->n_forced >= 0) {
      if (it >= st->n_forced) q.stop = 1;
      else q.b = st->forced[it];
    } else if (e <= st->tol) {
      q.stop = 1;
    } else if (it >= st->max_iter) {
      q.stop = 2;
    } else if (e <= st->e_hand) {
      q.stop = 5;
    } else if (st->stag && it - st->first >= 9 && e > st->recs[it - 2].e) {
      q.stop = 4;
    } else {
      q.b = dsq < dlin ? 0 : 1;
    }
    q.in = __hip_atomic_load(&st->recs[it].in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    q.out = wall_clock64();
    st->recs[it] = q;
    st->cur_b = q.b;
    st->ticket = 0;
    if (q.stop) st->stopped = 1;
    else st->it = it + 1;
    if (seen) {
      if (q.stop)
        __hip_atomic_store(&seen->stopped, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      else
        __hip_atomic_store(&seen->it, it + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

template <typename TI, typename TO>
__global__ void k_convert(const TI* __restrict__ in, TO* __restrict__ out, int64_t n, TO scale) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = i; p < n; p += stride) out[p] = (TO)in[p] * scale;
}

// The FP32 iterate made exactly symmetric in place: the split and FP32 squares compute both
// triangles only inside the 64 x 64 tiles on the diagonal of a block (everything else is
// computed once and mirrored), pairing the planes of an entry and of its transpose
// differently there, so X is symmetric only to rounding inside those tiles; the FP64
// refinement relies on symmetry.  Each such tile becomes (T + T^T)/2, formed in FP64 and
// rounded once (an entry and its transpose round the same sum).  One workgroup per diagonal
// tile, read once through LDS.
__global__ __launch_bounds__(256) void k_sym_diag(float* __restrict__ X,
                                                  const int64_t* __restrict__ offs,
                                                  const int32_t* __restrict__ npad) {
  __shared__ float t[64][65];
  const int s = blockIdx.y, b = blockIdx.x;
  const int np = npad[s];
  if (b * 64 >= np) return;  // the whole workgroup leaves together
  float* x = X + offs[s] + (int64_t)(b * 64) * np + b * 64;
  for (int e = threadIdx.x; e < 64 * 64; e += 256) t[e >> 6][e & 63] = x[(int64_t)(e >> 6) * np + (e & 63)];
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int r = e >> 6, c = e & 63;
    x[(int64_t)r * np + c] = (float)(0.5 * ((double)t[r][c] + (double)t[c][r]));
  }
}

// ---- scatter: column i of D = column (= row, X symmetric) j of its subgraph block -------
template <typename T>
__global__ __launch_bounds__(kT) void k_scatter(const T* __restrict__ X, const int64_t* __restrict__ offs,
                                                const int32_t* __restrict__ npad,
                                                const int32_t* __restrict__ sub_ptr,
                                                const int32_t* __restrict__ sub_idx,
                                                const int32_t* __restrict__ sub_pos,
                                                const int32_t* __restrict__ col_sub,
                                                const int32_t* __restrict__ col_loc, int w,
                                                int32_t* __restrict__ dcol, double* __restrict__ dval) {
  const int i = blockIdx.x;
  const int s = col_sub[i], j = col_loc[i];
  const int b = sub_ptr[s], n = sub_ptr[s + 1] - b, np = npad[s];
  const T* xr = X + offs[s] + (int64_t)j * np;
  int32_t* oc = dcol + (int64_t)i * w;
  double* ov = dval + (int64_t)i * w;
  for (int a = threadIdx.x; a < n; a += kT) {
    const int p = sub_pos[b + a];
    oc[p] = sub_idx[b + a];
    ov[p] = (double)xr[a];
  }
  for (int r = n + threadIdx.x; r < w; r += kT) {
    oc[r] = -1;
    ov[r] = 0.0;
  }
}

// max over core rows j < k_s and columns a < n_s of |S - X| (one block per subgraph)
template <typename T>
__global__ __launch_bounds__(kT) void k_idem(const T* __restrict__ X, const T* __restrict__ S,
                                             const int64_t* __restrict__ offs,
                                             const int32_t* __restrict__ npad,
                                             const int32_t* __restrict__ core_ptr,
                                             const int32_t* __restrict__ sub_ptr,
                                             double* __restrict__ out) {
  __shared__ double red[kT];
  const int s = blockIdx.x;
  const int np = npad[s], n = sub_ptr[s + 1] - sub_ptr[s], k = core_ptr[s + 1] - core_ptr[s];
  double m = 0.0;
  for (int64_t p = threadIdx.x; p < (int64_t)k * n; p += kT) {
    const int j = (int)(p / n), a = (int)(p - (int64_t)j * n);
    const int64_t q = offs[s] + (int64_t)j * np + a;
    m = fmax(m, fabs((double)S[q] - (double)X[q]));
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[s] = red[0];
}

// ---- core rows of a polynomial in X (FP64 refinement on the rows D keeps) -----------------
// A "row slab" holds k_s rows of width np_s per subgraph at soffs[s] (row stride np_s), the
// same layout as the first k_s rows of a block, so the trace, check and scatter kernels read a
// slab as they read a block.  Since X is symmetric, the core rows of q(X) are the transposed
// core columns, and V q(X) for a slab V needs only products V X.

// W = (scale V) X on the FP64 matrix cores (scale a power of two, applied exactly to V's entries
// as they are loaded: the stored iterate may be X / scale).  A workgroup computes all KMAX rows of
// 64 columns of W, its four waves a quarter of the reduction each (KMAX/16 x 4 tiles of 16 x 16
// per wave, v_mfma_f64_16x16x4, in chunks of 16 rows of X), added up through LDS in a fixed
// order.  Within a chunk, lane l (i = l%16, q = l/16) takes the four consecutive rows
// a + 4q + u, u = the MFMA index: its A operands of a row tile are one 32-byte run of V
// (V[16m + i][a + 4q .. a + 4q + 3]), and its B operands are 16-byte pairs of columns
// (X[a + 4q + u][c + 32g + 2i, +1]; tile 2g + h holds the columns of parity h of group g), so a
// chunk costs a wave 4 + 8 wide loads for 32 MFMAs.  X is read once; V (a few hundred KB per
// block) comes from L2: items lists a subgraph's column blocks on one XCD.  Rows of V beyond k_s
// are read in bounds (row k_s - 1) and zeroed by a select, keeping the loop free of branches.
// Output register r of lane l holds row 4r + q of its tile.
// Bound by the FP64 matrix cores and the reads of X together (N = 18000, 32 rows, FP32 X: 0.68 ms
// of products, 0.70 ms of reads at the copy rate), and by the latency of the reads: four waves per
// SIMD (128 registers) hide it better than the three that 151 registers leave (8 products 9.2
// against 9.9 ms).  Four waves on 64 columns are four times as many workgroups, a quarter as long,
// as a wave per 64 columns: no difference at N = 18000 (9.2 against 9.3 ms), but a chip that the
// small systems fill, N = 2050 2.13 -> 1.57 ms, N = 3000 (16 rows) 2.37 -> 1.7 ms.
// acc: y[q] (+)= c[q] W beside (or, with W NULL, instead of) W itself: the sums of a polynomial's
// terms as they appear.  stopped: the launch returns at once if *stopped is not 0.
struct RowsAcc {
  double* y[3];
  double c[3];
  int n, fresh;  // fresh: bit q set where y[q] starts here
};
template <int KMAX, typename TX>
__global__ __launch_bounds__(256, 4) void k_rows_mm(const TX* __restrict__ X,
                                                 const int64_t* __restrict__ offs,
                                                 const double* __restrict__ V,
                                                 double* __restrict__ W,
                                                 const int64_t* __restrict__ soffs,
                                                 const int32_t* __restrict__ core_ptr,
                                                 const int4* __restrict__ items, double scale,
                                                 RowsAcc sums,
                                                 const int32_t* __restrict__ stopped) {
  if (stopped && *stopped) return;
  using M = Mfma<double>;
  constexpr int MT = KMAX / 16, NT = 4, U = 4;
  __shared__ double2 red[2][MT * 2 * 4 * 64];
  const int4 it = items[blockIdx.x];
  if (it.x < 0) return;  // padding entry of an XCD queue
  const int s = it.x, np = it.w, cw = it.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k = core_ptr[s + 1] - core_ptr[s];
  const int i16 = lane & 15, kq = lane >> 4;
  M::acc_t acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = M::acc_t{0, 0, 0, 0};
  bool rows_in[MT];
  int64_t roff[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    rows_in[m] = m * 16 + i16 < k;
    roff[m] = (int64_t)min(m * 16 + i16, k - 1) * np;
  }
  const double* vb = V + soffs[s] + 4 * kq;
  const TX* xb = X + offs[s] + (int64_t)(4 * kq) * np + cw + 2 * i16;
  const int a_end = (wave + 1) * (np >> 2);  // np is a multiple of 64
  for (int a0 = wave * (np >> 2); a0 < a_end; a0 += 16) {
    double fa[U][MT], fb[U][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const double2* pv = reinterpret_cast<const double2*>(vb + roff[m] + a0);
      const double2 v0 = pv[0], v1 = pv[1];
      fa[0][m] = rows_in[m] ? v0.x * scale : 0.0;
      fa[1][m] = rows_in[m] ? v0.y * scale : 0.0;
      fa[2][m] = rows_in[m] ? v1.x * scale : 0.0;
      fa[3][m] = rows_in[m] ? v1.y * scale : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        if constexpr (std::is_same<TX, double>::value) {
          const double2 xv = *reinterpret_cast<const double2*>(xb + (int64_t)(a0 + u) * np + 32 * g);
          fb[u][2 * g] = xv.x;
          fb[u][2 * g + 1] = xv.y;
        } else {  // an FP32 X (exact in FP64): half the bytes per product
          const float2 xv = *reinterpret_cast<const float2*>(xb + (int64_t)(a0 + u) * np + 32 * g);
          fb[u][2 * g] = (double)xv.x;
          fb[u][2 * g + 1] = (double)xv.y;
        }
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = M::mma(fa[u][m], fb[u][n], acc[m][n]);
  }
  // the sum over the waves, (w0 + w2) + (w1 + w3): waves 2 and 3 hand theirs to 0 and 1, then
  // those exchange halves (two row tiles: a tile each; one: wave 0 takes all)
  auto put = [&](int buf, int m) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[buf][((m * 2 + g) * 4 + r) * 64 + lane] =
            double2{acc[m][2 * g][r], acc[m][2 * g + 1][r]};
  };
  auto add = [&](int buf, int m) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 v = red[buf][((m * 2 + g) * 4 + r) * 64 + lane];
        acc[m][2 * g][r] += v.x;
        acc[m][2 * g + 1][r] += v.y;
      }
  };
  if (wave >= 2)
#pragma unroll
    for (int m = 0; m < MT; ++m) put(wave - 2, m);
  __syncthreads();
  if (wave < 2)
#pragma unroll
    for (int m = 0; m < MT; ++m) add(wave, m);
  __syncthreads();
  if (wave == 1) put(0, 0);
  if (MT == 2 && wave == 0) put(1, MT - 1);
  __syncthreads();
  if (wave >= MT) return;
#pragma unroll
  for (int m = 0; m < MT; ++m)
    if (m == wave) add(m, m);
  const int64_t w0 = soffs[s] + cw + 2 * i16;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (m != wave) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = m * 16 + M::row(lane, r);
      if (j < k) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int64_t q = w0 + (int64_t)j * np + 32 * g;
          const double2 v = double2{acc[m][2 * g][r], acc[m][2 * g + 1][r]};
          if (W) *reinterpret_cast<double2*>(W + q) = v;
          for (int p = 0; p < sums.n; ++p) {
            double2* y = reinterpret_cast<double2*>(sums.y[p] + q);
            const double2 o = (sums.fresh >> p) & 1 ? double2{0.0, 0.0} : *y;
            *y = double2{o.x + sums.c[p] * v.x, o.y + sums.c[p] * v.y};
          }
        }
      }
    }
  }
}

// W = the first k_s rows of X (= E X for the core unit rows E), times scale (a power of two)
template <typename TX>
__global__ __launch_bounds__(256) void k_rows_copy(const TX* __restrict__ X,
                                                   const int64_t* __restrict__ offs,
                                                   const int32_t* __restrict__ npad,
                                                   double* __restrict__ W,
                                                   const int64_t* __restrict__ soffs,
                                                   const int32_t* __restrict__ core_ptr,
                                                   double scale) {
  const int s = blockIdx.y;
  const int np = npad[s], k = core_ptr[s + 1] - core_ptr[s];
  const int64_t n = (int64_t)k * np;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256)
    W[soffs[s] + p] = (double)X[offs[s] + p] * scale;
}

__global__ void k_max(const double* __restrict__ in, int n, double* __restrict__ out) {
  __shared__ double red[kT];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += kT) m = fmax(m, in[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}


// ---- adjoint kernels ------------------------------------------------------------------------
__global__ void k_fill(double* __restrict__ p, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = i; q < n; q += stride) p[q] = v;
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Gbar_K of every block from dL/dD on D's column-ELL pattern, symmetrised:
// Gbar[a][j] = (G(a, j) + G(j, a)) / 2 with G(a, j) = dL/dD[sub_a, sub_j] on core columns j.
__global__ __launch_bounds__(kT) void k_seed(const double* __restrict__ gval, int gw,
                                             const int32_t* __restrict__ core_ptr,
                                             const int32_t* __restrict__ sub_ptr,
                                             const int32_t* __restrict__ sub_idx,
                                             const int32_t* __restrict__ sub_pos,
                                             const int64_t* __restrict__ offs,
                                             const int32_t* __restrict__ npad,
                                             double* __restrict__ G) {
  const int s = blockIdx.x;
  const int b = sub_ptr[s], n = sub_ptr[s + 1] - b, k = core_ptr[s + 1] - core_ptr[s];
  const int np = npad[s];
  double* g = G + offs[s];
  for (int64_t p = threadIdx.x; p < (int64_t)n * k; p += kT) {
    const int a = (int)(p / k), j = (int)(p - (int64_t)a * k);
    double v = gval[(int64_t)sub_idx[b + j] * gw + sub_pos[b + a]];
    if (a < k) v += gval[(int64_t)sub_idx[b + a] * gw + sub_pos[b + j]];
    v *= 0.5;
    g[(int64_t)a * np + j] = v;
    if (a >= k) g[(int64_t)j * np + a] = v;
  }
}

// vertex -> subgraphs holding it: counts, fill, per-vertex sort by subgraph
__global__ void k_vs_count(const int32_t* __restrict__ sub_ptr, const int32_t* __restrict__ sub_idx,
                           int32_t* __restrict__ cnt) {
  const int s = blockIdx.x;
  for (int p = sub_ptr[s] + threadIdx.x; p < sub_ptr[s + 1]; p += blockDim.x)
    atomicAdd(&cnt[sub_idx[p]], 1);
}
__global__ void k_vs_fill(const int32_t* __restrict__ sub_ptr, const int32_t* __restrict__ sub_idx,
                          const int32_t* __restrict__ vs_ptr, int32_t* __restrict__ fill,
                          int32_t* __restrict__ vs_sub, int32_t* __restrict__ vs_loc) {
  const int s = blockIdx.x;
  for (int p = sub_ptr[s] + threadIdx.x; p < sub_ptr[s + 1]; p += blockDim.x) {
    const int v = sub_idx[p];
    const int q = vs_ptr[v] + atomicAdd(&fill[v], 1);
    vs_sub[q] = s;
    vs_loc[q] = p - sub_ptr[s];
  }
}
// The lists come in the order of the atomics; each vertex's is put in ascending order of the
// subgraphs (all different) by rank, a wave per vertex: a lane counts the entries below its own.
// (Sorted in place by a thread per vertex it took 423 us for 1800 lists of ~42; 6 us this way.)
__global__ __launch_bounds__(kT) void k_vs_sort(int n, const int32_t* __restrict__ vs_ptr,
                                                const int32_t* __restrict__ sub,
                                                const int32_t* __restrict__ loc,
                                                int32_t* __restrict__ vs_sub,
                                                int32_t* __restrict__ vs_loc) {
  const int v = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (v >= n) return;
  const int b = vs_ptr[v], e = vs_ptr[v + 1];
  for (int p = b + lane; p < e; p += 64) {
    const int key = sub[p];
    int rank = 0;
    for (int q = b; q < e; ++q) rank += sub[q] < key;
    vs_sub[b + rank] = key;
    vs_loc[b + rank] = loc[p];
  }
}

// dL/dH per ELL slot (i, j): sum over the subgraphs holding both i and j, ascending, of
// scale * Gbar_0[loc(i)][loc(j)]
__global__ void k_assemble(const int32_t* __restrict__ hcol, int n, int w,
                           const int32_t* __restrict__ vs_ptr, const int32_t* __restrict__ vs_sub,
                           const int32_t* __restrict__ vs_loc, const int64_t* __restrict__ offs,
                           const int32_t* __restrict__ npad, const double* __restrict__ G0,
                           double scale, double* __restrict__ gh) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)n * w) return;
  const int i = (int)(q / w);
  const int j = hcol[q];
  if ((unsigned)j >= (unsigned)n) {
    gh[q] = 0.0;
    return;
  }
  int pi = vs_ptr[i], ei = vs_ptr[i + 1], pj = vs_ptr[j], ej = vs_ptr[j + 1];
  double acc = 0.0;
  while (pi < ei && pj < ej) {
    const int si = vs_sub[pi], sj = vs_sub[pj];
    if (si < sj) ++pi;
    else if (sj < si) ++pj;
    else {
      const double g = G0[offs[si] + (int64_t)vs_loc[pi] * npad[si] + vs_loc[pj]];
      acc = acc + scale * g;
      ++pi;
      ++pj;
    }
  }
  gh[q] = acc;
}

int grid_for(int64_t n, int t, int cap = 1 << 20) {
  const int64_t b = (n + t - 1) / t;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

// ---- plan: padded sizes, offsets, tile lists ---------------------------------------------
// Square tiles are listed 128-edge tiles first, then 64-edge tiles; within each group the
// largest blocks come first (most k work per tile).
// Kernel variants of the batched products, one code per subgraph: 128 (128-edge tiles, two LDS
// stages), 64 (64-edge, two stages), 63 (64-edge, three stages), 62 (64-edge, two stages,
// register-staged loads), 32 (32-edge, k_square_small); split squares: 128 and 64, and for fp16
// planes 129 and 65 (128- and 64-edge tiles with the split under the products,
// k_symm_mm_split_il).
constexpr int kNVar = 7;
constexpr int kVariants[kNVar] = {128, 64, 63, 62, 129, 65, 32};
inline int variant_edge(int code) { return code >= 128 ? 128 : code == 32 ? 32 : 64; }
inline bool split_il_code(int code) { return code == 129 || code == 65; }
inline int variant_index(int code) {
  for (int v = 0; v < kNVar; ++v)
    if (kVariants[v] == code) return v;
  return -1;
}

// tiles per variant group (launch order as kVariants)
struct Groups {
  int n[kNVar] = {};
};

struct Plan {
  int n_sub = 0;
  std::vector<int32_t> npad;
  std::vector<int64_t> off;
  std::vector<int> bt;           // kernel variant code chosen for each subgraph
  int64_t total = 0;
  std::vector<int4> tiles;       // bi <= bj (symmetric products), grouped by variant
  Groups tg;                     //   (subgraph-major; per-subgraph launches use `ranges`)
  std::vector<int4> launch;      // the same tiles as launched in one batch, each variant group
  Groups lg;                     //   in XCD order
  std::vector<int4> ranges;      // per subgraph: first tile, tile count, variant code, s
  std::vector<int4> idem;        // 128-edge upper tiles covering the core rows (final check)
  double flops_alg = 0, flops_exec = 0;
  int max_npad = 0;
};

// XCD-aware order: the hardware hands workgroup b to XCD b % 8.  Whole subgraphs are dealt to
// the eight XCD queues (greedy, costliest first, onto the least loaded queue) and the queues
// are interleaved, so every tile of a subgraph runs on one XCD and its row panels stay in that
// XCD's L2.  Too few subgraphs to fill the queues evenly are cut where a queue is full instead
// (FP64 square of one block of 2048 rows 1171 -> 223 us, of two of 704 82 -> 43).  Queues are
// padded to equal length with empty entries (subgraph -1).
constexpr int kXcd = 8;

void xcd_order(std::vector<int4>& out, const std::vector<int4>& tiles,
               const std::vector<int4>& ranges, size_t r0, size_t r1) {
  if (r1 <= r0) return;
  std::vector<std::vector<int4>> q(kXcd);
  std::vector<double> load(kXcd, 0.0);
  for (size_t r = r0; r < r1; ++r) {
    const int4 rg = ranges[r];
    int best = 0;
    for (int x = 1; x < kXcd; ++x)
      if (load[x] < load[best]) best = x;
    for (int t = 0; t < rg.y; ++t) q[best].push_back(tiles[rg.x + t]);
    load[best] += (double)rg.y * tiles[rg.x].w;
  }
  const double total = std::accumulate(load.begin(), load.end(), 0.0);
  if (*std::max_element(load.begin(), load.end()) * kXcd > 1.25 * total) {
    for (auto& v : q) v.clear();
    double done = 0.0;
    for (size_t r = r0; r < r1; ++r)
      for (int t = 0; t < ranges[r].y; ++t) {
        const int4 tl = tiles[ranges[r].x + t];
        q[std::min(kXcd - 1, (int)(done * kXcd / total))].push_back(tl);
        done += tl.w;
      }
  }
  size_t len = 0;
  for (auto& v : q) len = std::max(len, v.size());
  const size_t base = out.size();
  out.resize(base + len * kXcd, make_int4(-1, 0, 0, 0));
  for (int x = 0; x < kXcd; ++x)
    for (size_t j = 0; j < q[x].size(); ++j) out[base + j * kXcd + x] = q[x][j];
}

Plan make_plan(const Part& P, const std::vector<int>* bt = nullptr, bool xcd = true) {
  Plan pl;
  pl.n_sub = P.n_sub;
  pl.npad.resize(P.n_sub);
  pl.off.resize(P.n_sub);
  pl.bt.assign(P.n_sub, kBT);
  if (bt) pl.bt = *bt;
  std::vector<int> order(P.n_sub);
  for (int s = 0; s < P.n_sub; ++s) {
    const int n = P.h_sub_ptr[s + 1] - P.h_sub_ptr[s];
    pl.npad[s] = padded(n);
    pl.off[s] = pl.total;
    pl.total += (int64_t)pl.npad[s] * pl.npad[s];
    pl.flops_alg += 2.0 * (double)n * n * n;
    pl.max_npad = std::max(pl.max_npad, pl.npad[s]);
    order[s] = s;
  }
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return pl.npad[a] > pl.npad[b]; });
  size_t r_first[kNVar + 1] = {};
  for (int v = 0; v < kNVar; ++v) {
    const int code = kVariants[v], edge = variant_edge(code);
    const int t0 = (int)pl.tiles.size();
    r_first[v] = pl.ranges.size();
    for (int s : order) {
      if (pl.bt[s] != code) continue;
      const int np = pl.npad[s], n = P.h_sub_ptr[s + 1] - P.h_sub_ptr[s];
      const int nb = (np + edge - 1) / edge;
      const int first = (int)pl.tiles.size();
      const int wt = edge / 2;  // wave tile edge (2 x 2 waves per tile)
      for (int bi = 0; bi < nb; ++bi)
        for (int bj = bi; bj < nb; ++bj) {
          pl.tiles.push_back(make_int4(s, bi, bj, n));
          // matrix-core work the tile executes: every wave whose block begins inside the n rows,
          // except the lower-left one of a diagonal tile, over k to the end of n's chunk
          for (int wr = 0; wr < 2; ++wr)
            for (int wc = 0; wc < 2; ++wc)
              if (bi * edge + wr * wt < n && bj * edge + wc * wt < n && !(bi == bj && wr > wc))
                pl.flops_exec += 2.0 * wt * wt * (double)((n + 31) / 32 * 32);
        }
      pl.ranges.push_back(make_int4(first, (int)pl.tiles.size() - first, code, s));
    }
    pl.tg.n[v] = (int)pl.tiles.size() - t0;
  }
  r_first[kNVar] = pl.ranges.size();
  // launch list of the batched squaring: each group in XCD order (or as listed)
  if (xcd) {
    for (int v = 0; v < kNVar; ++v) {
      const size_t before = pl.launch.size();
      xcd_order(pl.launch, pl.tiles, pl.ranges, r_first[v], r_first[v + 1]);
      pl.lg.n[v] = (int)(pl.launch.size() - before);
    }
  } else {
    pl.launch = pl.tiles;
    pl.lg = pl.tg;
  }
  for (int s : order) {
    const int n = P.h_sub_ptr[s + 1] - P.h_sub_ptr[s];
    const int nb = (pl.npad[s] + kBT - 1) / kBT;
    const int k = P.h_core_ptr[s + 1] - P.h_core_ptr[s];
    for (int bi = 0; bi < nb && bi * kBT < k; ++bi)
      for (int bj = bi; bj < nb; ++bj) pl.idem.push_back(make_int4(s, bi, bj, n));
  }
  return pl;
}

}  // namespace

struct TapeData {
  int N = 0, K = 0, stride = 4, max_sub = 0, max_core = 0;
  double emin = 0, emax = 0;
  std::vector<uint8_t> branch;
  Plan pl;
  DBuf<int64_t> offs;
  DBuf<int32_t> npad;
  DBuf<int4> tiles;
  DBuf<int32_t> core_ptr, sub_ptr, sub_idx, sub_pos;
  std::vector<CachedBuf> ckpt;  // X_0, X_stride, X_2stride, ...
  bool thins = false;           // stride 1 by the library's choice: fewer where they find no room
  void thin() {                 // to every fourth (nothing may read the others any more)
    std::vector<CachedBuf> kept;
    for (size_t i = 0; i < ckpt.size(); i += kThinned) kept.push_back(std::move(ckpt[i]));
    ckpt.swap(kept);
    stride = kThinned;
    thins = false;
  }
  static constexpr int kThinned = 4;
};
// Most memory of a tape that keeps every iterate because nobody asked for another stride: some
// thirty steps of 1 GiB.
constexpr size_t kTapeMost = (size_t)32 << 30;

namespace {

// One batched symmetric product over the variant groups of a tile list (see k_symm_mm).
template <typename T, int MODE>
void launch_symm(const T* A, const T* B, const T* E, T* out, T alpha, T beta, const int4* tiles,
                 const Groups& g, const int64_t* offs, hipStream_t s,
                 const int32_t* stopped = nullptr, int lin = 0,
                 const int32_t* lin_flag = nullptr) {
  if (g.n[4] > 0 || g.n[5] > 0) fail(GB_EHIP, "split-square tiles given to an FP64/FP32 product");
  const int4* t = tiles;
  if (g.n[0] > 0)
    hipLaunchKernelGGL((k_symm_mm<T, MODE, 128, 2>), dim3(g.n[0]), dim3(kT), 0, s, A, B, E, out,
                       alpha, beta, t, offs, stopped, lin, lin_flag, 0);
  t += g.n[0];
  if (g.n[1] > 0)
    hipLaunchKernelGGL((k_symm_mm<T, MODE, 64, 2>), dim3(g.n[1]), dim3(kT), 0, s, A, B, E, out,
                       alpha, beta, t, offs, stopped, lin, lin_flag, 0);
  t += g.n[1];
  if (g.n[2] > 0)
    hipLaunchKernelGGL((k_symm_mm<T, MODE, 64, 3>), dim3(g.n[2]), dim3(kT), 0, s, A, B, E, out,
                       alpha, beta, t, offs, stopped, lin, lin_flag, 0);
  t += g.n[2];
  if (g.n[3] > 0)
    hipLaunchKernelGGL((k_symm_mm<T, MODE, 64, 2, 1>), dim3(g.n[3]), dim3(kT), 0, s, A, B, E,
                       out, alpha, beta, t, offs, stopped, lin, lin_flag, 0);
  t += g.n[3];
  if (g.n[6] > 0) {
    if constexpr (MODE == 0)
      hipLaunchKernelGGL(k_square_small<T>, dim3(g.n[6]), dim3(kT), 0, s, A, out, t, offs, stopped,
                         lin, lin_flag);
    else
      fail(GB_EHIP, "32-edge tiles take squares only");
  }
  GB_LAUNCH_CHECK();
}

// One SP2 step on a tile list: the new iterate X^2 (lin = 0) or 2X - X^2 (lin = 1), or the
// branch read from *lin_flag on the device-driven loop.
template <typename T>
void launch_square(const T* X, T* S, const int4* tiles, const Groups& g, const int64_t* offs,
                   hipStream_t s, int lin = 0, const int32_t* stopped = nullptr,
                   const int32_t* lin_flag = nullptr) {
  launch_symm<T, 0>(X, X, X, S, (T)1, (T)0, tiles, g, offs, s, stopped, lin, lin_flag);
}

// a single group (the idempotency check's 128-edge tiles, one subgraph's range)
inline Groups one_group(int code, int count) {
  Groups g;
  g.n[variant_index(code)] = count;
  return g;
}

// the same with split squares (FP32 iterate X -> new FP32 iterate S; `planes` 1-3 bf16 planes
// or 4 = two fp16 planes), 128-edge tiles first, then 64-edge tiles
template <int NP, bool F16>
void launch_split_np(const float* X, float* S, const int4* tiles, const Groups& g,
                     const int64_t* offs, hipStream_t s, int lin, const int32_t* stopped,
                     const int32_t* lin_flag) {
  if (g.n[2] > 0 || g.n[3] > 0 || g.n[6] > 0)
    fail(GB_EHIP, "split squares take 128- or 64-edge tiles only");
  const int4* t = tiles;
  if (g.n[0] > 0)
    hipLaunchKernelGGL((k_symm_mm_split<NP, F16, 128>), dim3(g.n[0]), dim3(kT), 0, s, X, S, t,
                       offs, stopped, lin, lin_flag);
  t += g.n[0];
  if (g.n[1] > 0)
    hipLaunchKernelGGL((k_symm_mm_split<NP, F16, 64>), dim3(g.n[1]), dim3(kT), 0, s, X, S, t,
                       offs, stopped, lin, lin_flag);
  t += g.n[1];
  if (g.n[4] > 0 || g.n[5] > 0) {
    if constexpr (NP == 2 && F16) {
      if (g.n[4] > 0)
        hipLaunchKernelGGL(k_symm_mm_split_il<128>, dim3(g.n[4]), dim3(kT), 0, s, X, S, t, offs,
                           stopped, lin, lin_flag);
      t += g.n[4];
      if (g.n[5] > 0)
        hipLaunchKernelGGL(k_symm_mm_split_il<64>, dim3(g.n[5]), dim3(kT), 0, s, X, S, t, offs,
                           stopped, lin, lin_flag);
    } else {
      fail(GB_EHIP, "the interleaved split squares take fp16 planes only");
    }
  }
  GB_LAUNCH_CHECK();
}

void launch_split(const float* X, float* S, const int4* tiles, const Groups& g,
                  const int64_t* offs, hipStream_t s, int planes, int lin,
                  const int32_t* stopped = nullptr, const int32_t* lin_flag = nullptr) {
  if (planes == 1) launch_split_np<1, false>(X, S, tiles, g, offs, s, lin, stopped, lin_flag);
  else if (planes == 2) launch_split_np<2, false>(X, S, tiles, g, offs, s, lin, stopped, lin_flag);
  else if (planes == 4) launch_split_np<2, true>(X, S, tiles, g, offs, s, lin, stopped, lin_flag);
  else launch_split_np<3, false>(X, S, tiles, g, offs, s, lin, stopped, lin_flag);
}

// device tile table: the launch list, then (for launches per subgraph) the subgraph-major list
DBuf<int4> upload_tiles(const Plan& pl, hipStream_t s, bool per_subgraph) {
  DBuf<int4> t(pl.launch.size() + (per_subgraph ? pl.tiles.size() : 0), s);
  GB_HIP(hipMemcpyAsync(t.get(), pl.launch.data(), pl.launch.size() * sizeof(int4),
                        hipMemcpyHostToDevice, s));
  if (per_subgraph)
    GB_HIP(hipMemcpyAsync(t.get() + pl.launch.size(), pl.tiles.data(),
                          pl.tiles.size() * sizeof(int4), hipMemcpyHostToDevice, s));
  return t;
}

void launch_plan_square_f64(const double* X, double* S, const Plan& pl, const int4* tiles,
                            const int64_t* offs, hipStream_t s, int lin = 0) {
  launch_square<double>(X, S, tiles, pl.lg, offs, s, lin);
}

float elapsed(hipEvent_t a, hipEvent_t b) {
  float ms = 0.f;
  GB_HIP(hipEventElapsedTime(&ms, a, b));
  return ms;
}

struct PinnedRec {
  StepRec* h = nullptr;
  PinnedRec() { GB_HIP(hipHostMalloc((void**)&h, sizeof(StepRec), hipHostMallocDefault)); }
  ~PinnedRec() {
    if (h) (void)hipHostFree(h);
  }
};

// ---- autotuner: kernel variant of the split squares ------------------------------------------
// The first time a size class of batches is seen (tune_class; "bucket" in the table) for a kind of
// square (10 + planes; 0 FP64 and 1 FP32 take fixed variants), one squaring launch of the whole
// batch is timed with each kernel variant (one warm-up, two timed
// launches each) and the fastest is kept.  The table lives for the process and can be kept in
// a JSON file (gb_tune_save / gb_tune_load, or the GB_TUNE_FILE environment variable: read at
// the first tuning, rewritten after every new entry), tagged with the library's source hash and
// the device; a file with another tag is not used.
std::mutex g_tune_mu;
std::map<std::pair<int, int>, int> g_tune;  // (square kind, bucket) -> variant code
bool g_tune_env_read = false;

#ifndef GB_SOURCE_SHA
#define GB_SOURCE_SHA "unknown"
#endif

std::string tune_identity() {
  int dev = 0;
  GB_HIP(hipGetDevice(&dev));
  hipDeviceProp_t pr;
  GB_HIP(hipGetDeviceProperties(&pr, dev));
  char buf[512];
  snprintf(buf, sizeof(buf), "%s cu=%d %s", pr.gcnArchName, pr.multiProcessorCount, pr.name);
  for (char* c = buf; *c; ++c)
    if (*c == '"' || *c == '\\') *c = ' ';
  return buf;
}

// writes the table (caller holds g_tune_mu); false if the file cannot be written
bool tune_write(const char* path) {
  const std::string tmp = std::string(path) + ".tmp";
  FILE* f = fopen(tmp.c_str(), "w");
  if (!f) return false;
  fprintf(f, "{\"format\": \"libgb-tune-1\", \"library\": \"%s\", \"device\": \"%s\",\n \"entries\": [",
          GB_SOURCE_SHA, tune_identity().c_str());
  bool first = true;
  for (const auto& kv : g_tune) {
    fprintf(f, "%s\n  {\"kind\": %d, \"bucket\": %d, \"variant\": %d}", first ? "" : ",",
            kv.first.first, kv.first.second, kv.second);
    first = false;
  }
  fprintf(f, "]}\n");
  const bool ok = fclose(f) == 0;
  return ok && std::rename(tmp.c_str(), path) == 0;
}

// reads a table written by tune_write into g_tune (caller holds g_tune_mu); returns the number
// of entries, or -1 (message in *why) if the file is missing, malformed or for another library
// or device
int tune_read(const char* path, std::string* why) {
  FILE* f = fopen(path, "r");
  if (!f) {
    *why = "cannot open the file";
    return -1;
  }
  std::string txt;
  char chunk[4096];
  size_t got;
  while ((got = fread(chunk, 1, sizeof(chunk), f)) > 0) txt.append(chunk, got);
  fclose(f);
  auto field = [&](const char* key) -> std::string {
    const std::string k = std::string("\"") + key + "\": \"";
    const size_t a = txt.find(k);
    if (a == std::string::npos) return std::string("\x01");
    const size_t b = txt.find('"', a + k.size());
    return b == std::string::npos ? std::string("\x01") : txt.substr(a + k.size(), b - a - k.size());
  };
  if (field("format") != "libgb-tune-1") {
    *why = "not a libgb tuning table";
    return -1;
  }
  if (field("library") != GB_SOURCE_SHA) {
    *why = "written by another build of the library";
    return -1;
  }
  if (field("device") != tune_identity()) {
    *why = "written on another device";
    return -1;
  }
  std::map<std::pair<int, int>, int> t;
  size_t pos = 0;
  while ((pos = txt.find("{\"kind\":", pos)) != std::string::npos) {
    int kind, bucket, variant;
    if (sscanf(txt.c_str() + pos, "{\"kind\": %d, \"bucket\": %d, \"variant\": %d}", &kind,
               &bucket, &variant) != 3) {
      *why = "malformed entry";
      return -1;
    }
    // kinds: 0 FP64, 1 FP32, 10 + planes split squares; the interleaved split (129, 65)
    // exists for the fp16 planes (kind 14) only
    // (32 is chosen by the batch's size, never from a table)
    const bool known = variant_index(variant) >= 0 && variant != 32;
    const bool split = kind >= 11 && kind <= 14;
    const bool split_ok = variant == 128 || variant == 64 || (kind == 14 && split_il_code(variant));
    if (!known || bucket < 1 || !(kind == 0 || kind == 1 || split) || (split && !split_ok) ||
        (!split && split_il_code(variant))) {
      *why = "entry with an unknown kind, bucket or variant";
      return -1;
    }
    t[{kind, bucket}] = variant;
    pos += 8;
  }
  for (const auto& kv : t) g_tune[kv.first] = kv.second;
  return (int)t.size();
}

// the GB_TUNE_FILE table, read once (caller holds g_tune_mu; an unusable file is ignored)
void tune_env_read() {
  if (g_tune_env_read) return;
  g_tune_env_read = true;
  const char* path = std::getenv("GB_TUNE_FILE");
  std::string why;
  if (path && *path) (void)tune_read(path, &why);
}

void tune_env_write() {
  const char* path = std::getenv("GB_TUNE_FILE");
  if (path && *path) (void)tune_write(path);
}

// The size class of a batch in the tuning table: powers of two of its 128-edge tiles.
int tune_class(const Part& P) {
  int64_t t = 0;
  for (int q = 0; q < P.n_sub; ++q) {
    const int64_t nb = (padded(P.h_sub_ptr[q + 1] - P.h_sub_ptr[q]) + kBT - 1) / kBT;
    t += nb * (nb + 1) / 2;
  }
  int c = 1;
  while (((int64_t)1 << c) <= t) ++c;
  return c;
}

// The split squares' kernel for a batch: each variant timed on the whole batch, once per process
// and size class.  (One variant for all: a choice per size of block, each size timed by itself,
// paid for every variant's own launch and for small groups that cannot fill the device, which
// flattered small tiles: bf16 x 3 planes N = 2050 1.118 -> 1.032 ms a square, N = 6014 2.22 ->
// 2.11, fp16 N = 1400 0.341 -> 0.303, N = 2050 0.644 -> 0.633, N = 18000 3.88 -> 3.84.)
int tune_tiles(const Part& P, const float* X, float* S, const int64_t* offs, hipStream_t s, int kind,
               bool xcd, int planes) {
  const std::pair<int, int> key{kind, tune_class(P)};
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    tune_env_read();
    auto it = g_tune.find(key);
    if (it != g_tune.end()) return it->second;
  }
  Timer tm;
  int choice = 0;
  float best = INFINITY;
  for (int code : kVariants) {
    if (code != 128 && code != 64 && !(planes == 4 && split_il_code(code))) continue;
    const std::vector<int> bt(P.n_sub, code);
    const Plan pl = make_plan(P, &bt, xcd);
    DBuf<int4> tl = upload_tiles(pl, s, false);
    auto run = [&] { launch_split(X, S, tl.get(), pl.lg, offs, s, planes, 0); };
    run();
    GB_HIP(hipEventRecord(tm.a, s));
    run();
    run();
    GB_HIP(hipEventRecord(tm.b, s));
    GB_HIP(hipStreamSynchronize(s));
    const float ms = elapsed(tm.a, tm.b);
    if (ms < best) {
      best = ms;
      choice = code;
    }
  }
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune[key] = choice;
  tune_env_write();
  return choice;
}

// Squares on 32-edge tiles (k_square_small)?  FP64 while at most five 64-edge tiles fall to each of
// the 256 compute units, which is what one holds at a time: the launch then lasts as long as a
// tile does.  us on 64-edge -> 32-edge tiles: 1056 64-edge ones (2 blocks of 2048 rows) 367 -> 329,
// 1088 (8 of 1024) 191 -> 168, 1280 (128 of 256) 68.4 -> 53.6, but 1012 (4 of 1408) 202 -> 216.
// Past the line the gain falls with the reuse that small tiles give up: 1440 (12 of 900) 230 -> 186,
// 2024 (8 of 1408) 387 -> 407, 2400 (20 of 900) 371 -> 349, 3840 (32 of 900) 482 -> 468, 7680 (64 of
// 900) 924 -> 935.  FP32, whose products take half the time, up to one and a half: 325 (one of 1600)
// 72.5 -> 55.3, 396 (6 of 704) 35.3 -> 31.6, 400 (40 of 256) 17.7 -> 16.7; 448 (16 of 400) 23.7 ->
// 24.2, 640 (64 of 256) 21.8 -> 22.7.
template <typename T>
bool small_batch(const Part& P) {
  int64_t t64 = 0;
  for (int q = 0; q < P.n_sub; ++q) {
    const int64_t nb = padded(P.h_sub_ptr[q + 1] - P.h_sub_ptr[q]) / 64;
    t64 += nb * (nb + 1) / 2;
  }
  return t64 <= (std::is_same<T, double>::value ? 1280 : 400);
}

// The variant of every subgraph where a policy says it (0: split squares, timed).
template <typename T>
int fixed_tiles(const Part& P, int policy, int planes) {
  if (policy == 1) return kBT;
  if (policy == 2) return 64;
  if (policy == 4 && planes == 0) return 63;
  if (policy == 5 && planes == 0) return 62;
  if (policy == 6 && planes == 4) return 129;
  if (policy == 7 && planes == 4) return 65;
  // FP64 / FP32 squares: the register-staged 64-edge variant, the fastest measured in every
  // size bucket of the N = 1024, 18000 and 100000 systems (the others stay selectable), but for
  // small batches
  if (planes == 0) return small_batch<T>(P) ? 32 : 62;
  return 0;
}

// The tiles of a loop: pl and its device copy are made again where they are not of the variant
// asked for (tiles empty: not uploaded yet).
template <typename T>
void choose_tiles(const Part& P, Plan& pl, T* X, T* S, DBuf<int4>& tiles, const int64_t* offs,
                  hipStream_t s, int policy, int kind, gb_sp2_stats& st, bool xcd,
                  bool per_subgraph, int planes = 0, bool record = true) {
  int code = fixed_tiles<T>(P, policy, planes);
  if constexpr (std::is_same<T, float>::value) {
    if (!code) code = tune_tiles(P, X, S, offs, s, kind, xcd, planes);
  }
  const std::vector<int> bt(pl.n_sub, code);
  const bool changed = bt != pl.bt;
  if (changed) pl = make_plan(P, &bt, xcd);
  if (changed || !tiles.get()) tiles = upload_tiles(pl, s, per_subgraph);
  if (!record || policy == 1) return;  // the refinement's squares: the stats describe the loop's
  st.n_tile64 = 0;
  st.n_stage3 = 0;
  st.n_regstage = 0;
  st.n_split_il = 0;
  for (int e : bt) {
    st.n_split_il += split_il_code(e);
    st.n_tile64 += variant_edge(e) <= 64;
    st.n_stage3 += e == 63;
    st.n_regstage += e == 62 || e == 32;
  }
  st.square_flops_exec = pl.flops_exec;
}

// Decisions whose margin | |t2 - n| - |2 t1 - t2 - n| | is within the rounding of the summed
// traces (64 units in the last place of |t1| + |t2| + n_occ) could go the other way under
// another summation order; they are counted in the stats.
inline bool near_tie(const StepRec& r, double n_occ) {
  return r.margin <= 64.0 * 1.1102230246251565e-16 * (fabs(r.t1) + fabs(r.t2) + fabs(n_occ));
}

// Records of one step into the stats (it < 128).
inline void record_step(gb_sp2_stats& st, int it, const StepRec& r, bool applied, bool by_rule,
                        double n_occ) {
  if (it >= 128) return;
  st.t1[it] = r.t1;
  st.t2[it] = r.t2;
  st.idem = r.e;
  if (!applied) return;
  st.branch[it] = (uint8_t)r.b;
  if (by_rule) {
    st.min_margin = std::min(st.min_margin, r.margin);
    if (near_tie(r, n_occ)) ++st.n_near_tie;
  }
}

// One squaring launch of a step: the new iterate S = X^2 or 2X - X^2 (lin, or *lin_flag on the
// device-driven loops), batched over every subgraph or (per_subgraph) one launch per subgraph.
template <typename T>
void launch_step(const T* X, T* S, const Plan& pl, const int4* tiles, const int64_t* offs,
                 hipStream_t s, int planes, int lin, bool per_subgraph,
                 const int32_t* stopped = nullptr, const int32_t* lin_flag = nullptr) {
  const int nl = (int)pl.launch.size();
  if constexpr (std::is_same<T, float>::value) {
    if (planes > 0) {
      if (per_subgraph)
        for (const int4& rg : pl.ranges)
          launch_split(X, S, tiles + nl + rg.x, one_group(rg.z, rg.y), offs, s, planes, lin,
                       stopped, lin_flag);
      else
        launch_split(X, S, tiles, pl.lg, offs, s, planes, lin, stopped, lin_flag);
      return;
    }
  }
  if (per_subgraph)
    for (const int4& rg : pl.ranges)
      launch_square<T>(X, S, tiles + nl + rg.x, one_group(rg.z, rg.y), offs, s, lin, stopped,
                       lin_flag);
  else
    launch_square<T>(X, S, tiles, pl.lg, offs, s, lin, stopped, lin_flag);
}

// Host-driven SP2 loop in precision T on buffers X (current iterate) and S (scratch): each step
// takes the core traces of X and X^2 (from X), the FP64 decision, reads it back (one host round
// trip per step), then one squaring launch writes the next iterate.  Used for one launch per
// subgraph, for the tape of the adjoint and for the alternating FP64 refinement.  Returns the
// step index at which the stop rule fired, the replay ended, max_iter was reached, or (low
// precision) the idempotency error stagnated or fell to e_hand; X then holds the result.  first:
// the step at which a loop that goes on at it0 began (stagnation is judged over all of its steps).
template <typename T>
int sp2_loop(T*& X, T*& S, const Plan& pl, const DBuf<int4>& tiles, const int64_t* offs,
             const int32_t* npad, const Part& P, double n_occ, double tol, int max_iter,
             const uint8_t* branch_in, int n_branch_in, bool stagnation_stop, int it0,
             gb_sp2_stats& st, DBuf<StepRec>& recs, hipStream_t s, int* stop_kind,
             TapeData* tape = nullptr, int planes = 0, bool per_subgraph = false,
             bool alternate = false, double e_hand = 0.0, int first = -1) {
  Timer tm;
  PinnedRec pin;
  int it = it0;
  // the fp16 loop's iterate is stored as 2^14 X: its traces are scaled back
  const bool scaled = std::is_same<T, float>::value && planes == 4;
  const double ts1 = scaled ? kF16TraceDown1 : 1.0, ts2 = scaled ? kF16TraceDown2 : 1.0;
  T* const scratch[2] = {X, S};  // checkpoints are written where they stay, never over
  int prev_b = -1;
  std::vector<double> es;
  for (int q = first < 0 ? it0 : first; q < it0; ++q) es.push_back(fabs(st.t1[q] - st.t2[q]));
  DBuf<double> part(2 * (size_t)pl.n_sub, s);
  for (;;) {
    hipLaunchKernelGGL(k_trace_rows<T>, dim3(pl.n_sub), dim3(kT), 0, s, X, offs, npad,
                       P.core_ptr.get(), part.get(), nullptr, ts1, ts2);
    int forced = -1;
    if (branch_in) forced = it < n_branch_in ? (int)branch_in[it] : 2;
    else if (alternate && prev_b >= 0) forced = 10 + (1 - prev_b);
    const int at_max = it >= max_iter || it >= 127 ? 1 : 0;
    hipLaunchKernelGGL(k_decide, dim3(1), dim3(kT), 0, s, part.get(), pl.n_sub, n_occ, tol, forced,
                       at_max, recs.get());
    GB_LAUNCH_CHECK();
    GB_HIP(hipMemcpyAsync(pin.h, recs.get(), sizeof(StepRec), hipMemcpyDeviceToHost, s));
    GB_HIP(hipStreamSynchronize(s));
    const StepRec r = *pin.h;
    es.push_back(r.e);
    const bool hand = !r.stop && !branch_in && r.e <= e_hand;
    const bool stag = !r.stop && !hand && stagnation_stop && es.size() >= 10 &&
                      es.back() > es[es.size() - 3];
    record_step(st, it, r, !r.stop && !stag && !hand, branch_in == nullptr && !alternate, n_occ);
    if (r.stop) {
      *stop_kind = (r.stop == 1 && (branch_in == nullptr || r.e <= tol)) ? 1 : 2;
      if (branch_in && r.stop == 1) *stop_kind = r.e <= tol ? 1 : 3;
      return it;
    }
    if (stag || hand) {
      *stop_kind = hand ? 5 : 4;
      return it;
    }
    prev_b = r.b;
    T* to = nullptr;
    if constexpr (std::is_same<T, double>::value) {
      if (tape) {
        tape->branch.push_back((uint8_t)r.b);
        const size_t need = pl.total * sizeof(double);
        bool room = !tape->thins || (tape->ckpt.size() + 1) * need <= kTapeMost;
        if (room && (it + 1) % tape->stride == 0) {
          try {
            tape->ckpt.emplace_back(need, s);
            to = static_cast<double*>(tape->ckpt.back().p);
          } catch (const Error& e) {
            if (e.code != GB_ENOMEM || !tape->thins) throw;
            room = false;
          }
        }
        if (!room) {
          // X is a checkpoint, perhaps one of those that go
          if (X != scratch[0] && X != scratch[1]) {
            GB_HIP(hipMemcpyAsync(scratch[0], X, need, hipMemcpyDeviceToDevice, s));
            X = scratch[0];
            S = scratch[1];
          }
          GB_HIP(hipStreamSynchronize(s));
          tape->thin();
          if ((it + 1) % tape->stride == 0) {
            tape->ckpt.emplace_back(need, s);
            to = static_cast<double*>(tape->ckpt.back().p);
          }
        }
      }
    }
    if (!to) to = S;
    GB_HIP(hipEventRecord(tm.a, s));
    launch_step<T>(X, to, pl, tiles.get(), offs, s, planes, r.b == 1 ? 1 : 0, per_subgraph);
    GB_HIP(hipEventRecord(tm.b, s));
    X = to;
    S = X == scratch[0] ? scratch[1] : scratch[0];
    ++it;
    GB_HIP(hipEventSynchronize(tm.b));
    if (std::is_same<T, float>::value) {
      st.ms_square_lo += elapsed(tm.a, tm.b);
      st.n_square_lo += 1;
    } else {
      st.ms_square += elapsed(tm.a, tm.b);
      st.n_square += 1;
    }
  }
}

// The progress words of one device-driven loop.
struct ProgressLease {
  LoopProgress* p = nullptr;
  int dev = 0;
  ProgressLease() {
    GB_HIP(hipGetDevice(&dev));
    if (!pool().take(dev, &p))
      GB_HIP(hipHostMalloc((void**)&p, sizeof(LoopProgress), hipHostMallocDefault));
  }
  ProgressLease(const ProgressLease&) = delete;
  ProgressLease& operator=(const ProgressLease&) = delete;
  ~ProgressLease() {
    wait_if_failing();  // the loop's kernels write it
    if (p && !pool().give(dev, p)) (void)hipHostFree(p);
  }

  static IdlePool<LoopProgress*>& pool() {
    static auto* q = new IdlePool<LoopProgress*>;
    return *q;
  }
};

}  // namespace

void progress_trim() {
  ProgressLease::pool().drain([](LoopProgress* p) { (void)hipHostFree(p); });
}

namespace {

double wall_clock_khz() {
  thread_local std::map<int, int> rate;
  int dev = 0;
  GB_HIP(hipGetDevice(&dev));
  int& r = rate[dev];
  if (!r) GB_HIP(hipDeviceGetAttribute(&r, hipDeviceAttributeWallClockRate, dev));
  return r;
}

__global__ void k_loop_init(LoopState* __restrict__ st, LoopInit in) {
  st->it = in.it0;
  st->first = in.first;
  for (int i = 1; i <= 2; ++i)
    if (in.it0 - i >= in.first) st->recs[in.it0 - i].e = in.e_back[i - 1];
  st->stopped = 0;
  st->max_iter = in.max_iter;
  st->n_forced = in.n_forced;
  st->stag = in.stag;
  st->cur_b = -1;
  st->n_occ = in.n_occ;
  st->tol = in.tol;
  st->e_hand = in.e_hand;
  st->ticket = 0;
  for (int i = 0; i < 128; ++i) st->forced[i] = in.forced[i];
}

// Device-driven SP2 loop (launch modes 0 and 2): the stop flag, the step counter, the branch
// and the step records live on the device, each squaring launch reads the branch there, and
// every kernel of a step returns at once after the stop, so steps are enqueued without waiting
// for any decision.  Mode 0 keeps kAhead steps in the queue beyond the last decision, which the
// kernels post to pinned memory (32 steps enqueued at once left 15 empty ones behind the stop, 20
// us each at N = 2050, and an event before and after every square: 45 us a step at 256 orbitals,
// where the square takes 11).  Mode 2 captures two steps, one per buffer parity, in a hipGraph and
// replays it, 32 steps and then 8 at a time, reading the loop state in between.
template <typename T>
int sp2_loop_dev(T*& X, T*& S, const Plan& pl, const DBuf<int4>& tiles, const int64_t* offs,
                 const int32_t* npad, const Part& P, double n_occ, double tol, int max_iter,
                 const uint8_t* branch_in, int n_branch_in, bool stagnation_stop, int it0,
                 gb_sp2_stats& st, hipStream_t s, int* stop_kind, int planes, bool graph,
                 double e_hand = 0.0, int first = -1) {
  constexpr int kFirst = 32, kMore = 8, kAhead = 4;
  // index of the last decision the loop can reach: it stops there at the latest
  const int last = branch_in ? std::min(n_branch_in, 127) : std::min(max_iter, 127);
  if (last < it0) fail(GB_EINVAL, "no SP2 step left (first step %d, last %d)", it0, last);
  const int max_dec = last - it0 + 1;
  LoopInit in{};
  in.it0 = it0;
  in.first = first < 0 ? it0 : first;
  for (int i = 1; i <= 2; ++i)
    in.e_back[i - 1] = it0 - i >= in.first ? fabs(st.t1[it0 - i] - st.t2[it0 - i]) : 0.0;
  in.max_iter = max_iter;
  in.n_forced = branch_in ? std::min(n_branch_in, 127) : -1;
  in.stag = stagnation_stop ? 1 : 0;
  in.n_occ = n_occ;
  in.tol = tol;
  in.e_hand = e_hand;
  if (branch_in) std::memcpy(in.forced, branch_in, std::min(n_branch_in, 128));
  DBuf<LoopState> d(1, s);
  DBuf<double> part(2 * (size_t)pl.n_sub, s);
  // the fp16 loop's iterate is stored as 2^14 X: its traces are scaled back
  const bool scaled = std::is_same<T, float>::value && planes == 4;
  const double ts1 = scaled ? kF16TraceDown1 : 1.0, ts2 = scaled ? kF16TraceDown2 : 1.0;
  hipLaunchKernelGGL(k_loop_init, dim3(1), dim3(1), 0, s, d.get(), in);
  GB_LAUNCH_CHECK();
  const int32_t* stopped = &d.get()->stopped;
  const int32_t* cur_b = &d.get()->cur_b;
  std::unique_ptr<ProgressLease> progress(graph ? nullptr : new ProgressLease);
  LoopProgress* const seen = graph ? nullptr : progress->p;
  auto enqueue = [&](hipStream_t q, int k) {  // step k of the loop (0-based)
    T* A = (k & 1) ? S : X;
    T* B = (k & 1) ? X : S;
    hipLaunchKernelGGL(k_trace_step<T>, dim3(pl.n_sub), dim3(kT), 0, q, A, offs, npad,
                       P.core_ptr.get(), part.get(), ts1, ts2, d.get(), seen);
    GB_LAUNCH_CHECK();
    launch_step<T>(A, B, pl, tiles.get(), offs, q, planes, 0, false, stopped, cur_b);
  };
  hipStream_t cs = nullptr;
  hipGraph_t gr = nullptr;
  hipGraphExec_t exec = nullptr;
  struct Cleanup {
    hipStream_t& cs;
    hipGraph_t& g;
    hipGraphExec_t& e;
    ~Cleanup() {
      if (e) (void)hipGraphExecDestroy(e);
      if (g) (void)hipGraphDestroy(g);
      if (cs) (void)hipStreamDestroy(cs);
    }
  } cleanup{cs, gr, exec};
  if (graph) {
    GB_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    GB_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    enqueue(cs, 0);
    enqueue(cs, 1);
    GB_HIP(hipStreamEndCapture(cs, &gr));
    GB_HIP(hipGraphInstantiate(&exec, gr, nullptr, nullptr, 0));
  }
  LoopState h;
  int queued = 0;
  if (seen) {
    auto word = [](int32_t& w) { return __atomic_load_n(&w, __ATOMIC_RELAXED); };
    __atomic_store_n(&seen->it, it0, __ATOMIC_RELAXED);
    __atomic_store_n(&seen->stopped, 0, __ATOMIC_RELAXED);
    int idle = 0;  // looks since the last step was enqueued
    while (queued < max_dec && !word(seen->stopped)) {
      if (queued < word(seen->it) - it0 + kAhead) {
        enqueue(s, queued++);
        idle = 0;
        continue;
      }
      // a step of 0.1 ms or less is waited for awake; longer ones leave time to sleep, since the
      // queue holds several (and now and then the stream is asked whether it still runs)
      if (++idle <= (1 << 15)) continue;
      std::this_thread::sleep_for(std::chrono::microseconds(20));
      if (idle % 64 == 0) {
        const hipError_t e = hipStreamQuery(s);
        if (e == hipSuccess) break;  // nothing is left in the queue: the state tells
        if (e != hipErrorNotReady) GB_HIP(e);
        (void)hipGetLastError();  // "not ready" is no error of the launches that follow
      }
    }
  }
  for (;;) {
    if (graph) {
      const int batch = std::min(queued == 0 ? kFirst : kMore, max_dec - queued);
      const int pairs = (batch + 1) / 2;  // the graph holds two steps
      for (int r = 0; r < pairs; ++r) GB_HIP(hipGraphLaunch(exec, s));
      queued += 2 * pairs;
    }
    GB_HIP(hipMemcpyAsync(&h, d.get(), sizeof(h), hipMemcpyDeviceToHost, s));
    GB_HIP(hipStreamSynchronize(s));
    if (h.stopped) break;
    if (queued >= max_dec) fail(GB_EHIP, "device-driven SP2 loop did not stop");
    if (!graph)
      for (int k = 0; k < kMore && queued < max_dec; ++k) enqueue(s, queued++);
  }
  const int it_stop = h.it;
  for (int it = it0; it <= it_stop && it < 128; ++it)
    record_step(st, it, h.recs[it], it < it_stop, branch_in == nullptr, n_occ);
  const int n_sq = it_stop - it0;
  double ticks = 0.0;
  for (int it = it0; it < it_stop && it + 1 < 128; ++it)
    ticks += (double)std::max(0ll, h.recs[it + 1].in - h.recs[it].out);
  const float ms = graph ? 0.f : (float)(ticks / wall_clock_khz());
  if (std::is_same<T, float>::value) {
    st.n_square_lo += n_sq;
    st.ms_square_lo += ms;
  } else {
    st.n_square += n_sq;
    st.ms_square += ms;
  }
  const StepRec& lr = h.recs[it_stop];
  if (lr.stop == 1) *stop_kind = (branch_in && lr.e > tol) ? 3 : 1;
  else *stop_kind = lr.stop == 4 || lr.stop == 5 ? lr.stop : 2;
  // n_sq squares were applied, each moving the iterate to the other buffer
  if (n_sq % 2 == 1) std::swap(X, S);
  return it_stop;
}

}  // namespace

// ---- FP64 refinement on the core rows -------------------------------------------------------
// D keeps only the core columns of each block, i.e. (X symmetric) its core rows E q(X) for the
// core unit rows E, and E X^j takes one slab product (2 n^2 k flops instead of 2 n^3) from
// E X^{j-1}.  The refinement evaluates q = S_m, the polynomial of degree 2m - 1 that is flat to
// order m at 0 and 1 (S_2 = 3x^2 - 2x^3 is McWeeny's), so an eigenvalue off by d ends
// C(2m-1, m) d^m off: the terms m .. 2m - 1 of S_m are added up as the powers appear, the FP64
// stop test is taken on each S_m in turn, and the launches after the first that passes return
// at once.  The order in which S_2 twice (degree 9, 8 products, 27 d^4) does it needs 6 products
// (S_4: 35 d^4), and 8 give 126 d^5 (S_5).
constexpr int kSmoothMax = 6;

// coefficient of x^j in S_m, m <= j < 2m: (-1)^i C(m-1+i, i) C(2m-1, m-1-i) with i = j - m
double smooth_coef(int m, int j) {
  auto binom = [](int n, int k) {
    double b = 1.0;
    for (int i = 1; i <= k; ++i) b = b * (n - k + i) / i;
    return b;
  };
  const int i = j - m;
  const double c = std::rint(binom(m - 1 + i, i)) * std::rint(binom(2 * m - 1, m - 1 - i));
  return i % 2 ? -c : c;
}

// The idempotency measure at which the low-precision loop hands over to S_6: one eigenvalue
// carrying all of e ends C(11, 6) e^6 = 462 e^6 off, which is the tolerance here.  (Its own squares
// cost 3.7 ms at N = 18000, two more slab products 2.3 ms, and a square at this stage gains at most
// one order; beyond this point it also runs into its rounding floor.)
double handover_measure(double tol) { return std::pow(tol / 462.0, 1.0 / 6.0); }

// Stop flag and last record of the refinement's checks (device-driven, as LoopState): done is 0,
// or the order m of the S_m that passed (1: the iterate itself).
struct RefineState {
  int32_t done, pad;
  StepRec rec;
};

__global__ __launch_bounds__(kT) void k_refine_check(const double* __restrict__ part, int n_sub,
                                                     double n_occ, double thr, int m,
                                                     RefineState* __restrict__ st) {
  if (st->done) return;
  double t1, t2;
  sum_partials(part, n_sub, &t1, &t2);
  if (threadIdx.x == 0) {
    const double e = fabs(t1 - t2);
    StepRec q;
    q.t1 = t1;
    q.t2 = t2;
    q.e = e;
    q.margin = fabs(fabs(t2 - n_occ) - fabs(2.0 * t1 - t2 - n_occ));
    q.b = -1;
    q.stop = 1;
    q.pad0 = q.pad1 = 0;
    st->rec = q;
    if (e <= thr) st->done = m;
  }
}

struct CoreRows {
  int kmax = 0;
  int64_t total = 0;  // doubles per slab
  std::vector<int64_t> so;  // slab offset of each subgraph (host)
  std::vector<int4> items;  // (subgraph, first column, -, npad) of every 64 columns of a slab
  DBuf<int64_t> soffs;      // so and items on the device
  DBuf<int4> ditems;
};

// host part: the slab layout (false when a core exceeds 32 rows: whole blocks instead)
bool core_rows_sizes(const Part& P, const Plan& pl, CoreRows& cr) {
  int kmax = 0;
  for (int q = 0; q < pl.n_sub; ++q) {
    kmax = std::max(kmax, P.h_core_ptr[q + 1] - P.h_core_ptr[q]);
    if (pl.npad[q] % 64) return false;
  }
  if (kmax > 32) return false;
  cr.so.resize(pl.n_sub);
  int64_t t = 0;
  for (int q = 0; q < pl.n_sub; ++q) {
    cr.so[q] = t;
    t += (int64_t)(P.h_core_ptr[q + 1] - P.h_core_ptr[q]) * pl.npad[q];
  }
  cr.kmax = kmax <= 16 ? 16 : 32;
  cr.total = std::max<int64_t>(t, 1);
  return true;
}

bool core_rows_plan(const Part& P, const Plan& pl, CoreRows& cr, hipStream_t s) {
  if (!core_rows_sizes(P, pl, cr)) return false;
  // 64 columns per workgroup, largest blocks first, a subgraph's on one XCD
  std::vector<int> order(pl.n_sub);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return pl.npad[a] > pl.npad[b]; });
  std::vector<int4> list, ranges;
  for (int q : order) {
    const int first = (int)list.size();
    for (int c = 0; c < pl.npad[q]; c += 64) list.push_back(make_int4(q, c, 0, pl.npad[q]));
    ranges.push_back(make_int4(first, (int)list.size() - first, 0, q));
  }
  xcd_order(cr.items, list, ranges, 0, ranges.size());
  cr.soffs = DBuf<int64_t>(pl.n_sub, s);
  cr.ditems = DBuf<int4>(cr.items.size(), s);
  // cr's vectors live as long as cr, so the copies need no wait
  GB_HIP(hipMemcpyAsync(cr.soffs.get(), cr.so.data(), pl.n_sub * 8, hipMemcpyHostToDevice, s));
  GB_HIP(hipMemcpyAsync(cr.ditems.get(), cr.items.data(), cr.items.size() * sizeof(int4),
                        hipMemcpyHostToDevice, s));
  return true;
}

struct RowsCtx {
  const CoreRows& cr;
  const Plan& pl;
  const Part& P;
  const int64_t* offs;
  const int32_t* npad;
  hipStream_t s;
  double xscale;  // the stored iterate is X / xscale
  template <typename TX>
  void mm(const TX* X, const double* V, double* W, const RowsAcc& sums = RowsAcc{},
          const int32_t* stopped = nullptr) const {
    const dim3 grid(cr.items.size());
    if (cr.kmax == 16)
      hipLaunchKernelGGL((k_rows_mm<16, TX>), grid, dim3(256), 0, s, X, offs, V, W,
                         cr.soffs.get(), P.core_ptr.get(), cr.ditems.get(), xscale, sums, stopped);
    else
      hipLaunchKernelGGL((k_rows_mm<32, TX>), grid, dim3(256), 0, s, X, offs, V, W,
                         cr.soffs.get(), P.core_ptr.get(), cr.ditems.get(), xscale, sums, stopped);
    GB_LAUNCH_CHECK();
  }
};

int tune_save(const char* path) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  tune_env_read();
  if (!tune_write(path)) return -1;
  return (int)g_tune.size();
}

int tune_load(const char* path, std::string* why) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune_env_read = true;  // an explicit table replaces the environment's
  return tune_read(path, why);
}

void density_slots(const Part& P, int n, int width, const gb_sp2_opts& o,
                   size_t bytes[Workspace::kSlots]) {
  for (int i = 0; i < Workspace::kSlots; ++i) bytes[i] = 0;
  const Plan pl = make_plan(P, nullptr, o.tile_order == 0);
  const size_t t = (size_t)pl.total;
  bytes[0] = bytes[1] = t * 8;  // FP64 X, S
  if (o.precision != GB_FP64) {
    bytes[2] = t * 8;             // FP64 McWeeny product (whole-block refinement)
    bytes[3] = bytes[4] = t * 4;  // FP32 X, S
    CoreRows cr;
    if (core_rows_sizes(P, pl, cr)) bytes[7] = 5 * (size_t)cr.total * 8;  // core-row slabs
  }
  bytes[8] = (size_t)n * width * 8;  // X0 on H's pattern
}

void density(const gb_ell& H, int32_t n_occ, const gb_sp2_opts& o, const Part& P, double emin,
             double emax, const double* x0, gb_ell& D, gb_sp2_stats& st, hipStream_t s,
             TapeData** tape_out, Workspace* ext) {
  Timer t_all;
  GB_HIP(hipEventRecord(t_all.a, s));
  const bool xcd = o.tile_order == 0;
  DBuf<StepRec> recs(2, s);
  const int N = H.n;
  const double tol = o.idem_tol > 0 ? o.idem_tol : 1e-10 * N / 1024.0;
  const int max_iter = o.max_iter > 0 ? o.max_iter : 100;
  const bool low = o.precision != GB_FP64;
  // bf16 planes of the low-precision square: 0 = native FP32 MFMA
  // split planes of the low-precision square: 0 = native FP32 MFMA; 1 / 2 / 3 bf16 planes;
  // 4 = two fp16 planes
  const int planes = o.precision == GB_BF16_REFINE ? 1 : o.precision == GB_BF16X3_REFINE ? 2
                   : o.precision == GB_BF16X6_REFINE ? 3 : o.precision == GB_FP16X3_REFINE ? 4
                   : 0;
  const int nhi = low ? std::min(std::max(0, o.n_fp64_first), max_iter) : 0;
  // the plan of the first loop, where its tiles are known (FP64 steps before a low-precision loop:
  // 128-edge tiles); offsets and padded sizes go up in one copy, the tiles when a loop takes them
  const int code0 = nhi > 0 ? kBT
                    : low   ? fixed_tiles<float>(P, o.tile_policy, planes)
                            : fixed_tiles<double>(P, o.tile_policy, 0);
  const std::vector<int> bt0(P.n_sub, code0 ? code0 : kBT);
  Plan pl = make_plan(P, &bt0, xcd);
  st.square_flops = pl.flops_alg;
  st.square_flops_exec = pl.flops_exec;
  std::vector<int64_t> sizes(pl.off);
  sizes.resize(pl.n_sub + ((size_t)pl.n_sub + 1) / 2);
  std::memcpy(sizes.data() + pl.n_sub, pl.npad.data(), pl.n_sub * sizeof(int32_t));
  DBuf<int64_t> dsizes(sizes.size(), s);
  GB_HIP(hipMemcpyAsync(dsizes.get(), sizes.data(), sizes.size() * 8, hipMemcpyHostToDevice, s));
  const int64_t* const offs = dsizes.get();
  const int32_t* const npad = reinterpret_cast<const int32_t*>(dsizes.get() + pl.n_sub);
  DBuf<int4> tiles;
  const int n_refine = o.n_refine;
  const bool per_sub = o.launch_mode == 1;
  // launch modes 0 (default) and 2 run the loop on the device; 1 (one launch per subgraph) and
  // 3 read every decision back on the host
  const bool dev_loop = o.launch_mode == 0 || o.launch_mode == 2;
  int stop_kind = 0;
  // stage timings: events read once the call has finished its work (no wait per stage)
  Timer t_gather, t_sp2, t_ref, t_scat;
  // the gather is timed with the first buffer allocation included
  GB_HIP(hipEventRecord(t_gather.a, s));
  const size_t lds_g = (size_t)pl.max_npad * 8 + (size_t)P.max_sub * 4 + 64;
  if (lds_g > 160 * 1024) fail(GB_EUNSUPPORTED, "subgraph of %d vertices too large", P.max_sub);
  const dim3 ggrid(pl.n_sub, (pl.max_npad + kRows - 1) / kRows);
  // batch buffers from the cached workspace or the caller's: slots 0-2 FP64 (X, S, McWeeny
  // T), 3-4 FP32, 7 the core-row slabs
  WsLease ws(ext);
  double* const X64 = ws->get<double>(0, pl.total, s);
  double* const S64 = ws->get<double>(1, pl.total, s);
  double* xd = X64;
  double* sd = S64;
  int it_end = 0;
  bool done = false;  // the FP64 steps before a low-precision loop already converged
  // After a low-precision loop: its iterate made exactly symmetric in FP32 (what the core-row
  // refinement reads; stored as X / xs_scale, the fp16 loop's 2^14 X), and an FP64 copy of X
  // in xd only where whole blocks are refined, checked or scattered (ensure_xd).
  const float* xs = nullptr;
  double xs_scale = 1.0;
  bool xd_ready = true;
  std::function<void(double)> run_low;  // the low-precision loop from step it_end on
  if (low) {
    float* xf = ws->get<float>(3, pl.total, s);
    float* sf = ws->get<float>(4, pl.total, s);
    if (nhi > 0) {
      hipLaunchKernelGGL(k_gather<double>, ggrid, dim3(kT), lds_g, s, H.col, x0, H.width,
                         P.core_ptr.get(), P.sub_ptr.get(), P.sub_idx.get(), offs,
                         npad, xd, 1.0);
    } else {
      hipLaunchKernelGGL(k_gather<float>, ggrid, dim3(kT), lds_g, s, H.col, x0, H.width,
                         P.core_ptr.get(), P.sub_ptr.get(), P.sub_idx.get(), offs,
                         npad, xf, planes == 4 ? kF16Scale : 1.0f);
    }
    GB_LAUNCH_CHECK();
    GB_HIP(hipEventRecord(t_gather.b, s));
    GB_HIP(hipEventRecord(t_sp2.a, s));
    if (nhi > 0) {
      tiles = upload_tiles(pl, s, per_sub);
      // the first steps, where the spectral gap of X is smallest and rounding errors are
      // amplified most, in FP64
      if (dev_loop)
        it_end = sp2_loop_dev<double>(xd, sd, pl, tiles, offs, npad, P, n_occ, tol, nhi,
                                      o.branch_in, o.n_branch_in, false, 0, st, s, &stop_kind, 0,
                                      o.launch_mode == 2);
      else
        it_end = sp2_loop<double>(xd, sd, pl, tiles, offs, npad, P, n_occ, tol, nhi, o.branch_in,
                                  o.n_branch_in, false, 0, st, recs, s, &stop_kind, nullptr, 0,
                                  per_sub);
      done = stop_kind == 1 || stop_kind == 3;
      if (!done) {
        hipLaunchKernelGGL((k_convert<double, float>), dim3(grid_for(pl.total, kT, 65536)),
                           dim3(kT), 0, s, xd, xf, pl.total, planes == 4 ? kF16Scale : 1.0f);
        GB_LAUNCH_CHECK();
      }
    }
    if (!done) {
      st.planes_db = planes;
      // The low-precision loop hands over to the refinement as soon as that finishes the job
      // (a replayed sequence or a given number of steps runs as asked).  Where the refinement
      // is by other means, and where it did not finish the job, the loop runs until its own
      // rounding floor (the stagnation stop) unless the traces already agree to 1e-7 per 1024
      // orbitals.
      CoreRows sizes;
      const bool by_rows = o.refine_kind != 1 && n_refine == 0 && !o.branch_in &&
                           core_rows_sizes(P, pl, sizes);
      run_low = [&, xf, sf, first = it_end](double e_hand) mutable {
        const double tol_lo = 1e-7 * N / 1024.0;
        // FP32 squares: kind 1; split squares: kind 10 + planes (128- or 64-edge tiles)
        choose_tiles<float>(P, pl, xf, sf, tiles, offs, s, o.tile_policy,
                            planes ? 10 + planes : 1, st, xcd, per_sub, planes);
        if (dev_loop)
          it_end = sp2_loop_dev<float>(xf, sf, pl, tiles, offs, npad, P, n_occ, tol_lo, max_iter,
                                       o.branch_in, o.n_branch_in, true, it_end, st, s, &stop_kind,
                                       planes, o.launch_mode == 2, e_hand, first);
        else
          it_end = sp2_loop<float>(xf, sf, pl, tiles, offs, npad, P, n_occ, tol_lo, max_iter,
                                   o.branch_in, o.n_branch_in, true, it_end, st, recs, s,
                                   &stop_kind, nullptr, planes, per_sub, false, e_hand, first);
        // continue from X made exactly symmetric, in FP32, in place (every block is padded to a
        // multiple of 64)
        hipLaunchKernelGGL(k_sym_diag, dim3(pl.max_npad / 64, pl.n_sub), dim3(256), 0, s, xf,
                           offs, npad);
        GB_LAUNCH_CHECK();
        xs = xf;
        xd_ready = false;
      };
      run_low(by_rows ? handover_measure(tol) : 0.0);
      xs_scale = planes == 4 ? (double)kF16Down : 1.0;
    }
    GB_HIP(hipEventRecord(t_sp2.b, s));
  } else {
    choose_tiles<double>(P, pl, xd, sd, tiles, offs, s, o.tile_policy, 0, st, xcd,
                         per_sub);
    hipLaunchKernelGGL(k_gather<double>, ggrid, dim3(kT), lds_g, s, H.col, x0, H.width,
                       P.core_ptr.get(), P.sub_ptr.get(), P.sub_idx.get(), offs, npad,
                       X64, 1.0);
    GB_LAUNCH_CHECK();
    if (tape_out) {
      TapeData* t = new TapeData();
      *tape_out = t;
      t->N = N;
      t->emin = emin;
      t->emax = emax;
      // every iterate where some thirty of them are small change in HBM (the reverse sweep then
      // recomputes nothing), else, and from where they find no room on, every fourth
      t->stride = o.tape_stride > 0 ? o.tape_stride
                  : 32 * (size_t)pl.total * 8 <= kTapeMost ? 1 : TapeData::kThinned;
      t->thins = o.tape_stride <= 0 && t->stride == 1;
      t->max_sub = P.max_sub;
      for (int q = 0; q < P.n_sub; ++q)
        t->max_core = std::max(t->max_core, P.h_core_ptr[q + 1] - P.h_core_ptr[q]);
      const std::vector<int> bt(P.n_sub, 62);  // the reverse sweep's tiles, whatever the policy
      t->pl = make_plan(P, &bt, xcd);
      auto dup_i32 = [&](DBuf<int32_t>& dst, const DBuf<int32_t>& src, size_t n) {
        dst = DBuf<int32_t>(n, nullptr);
        GB_HIP(hipMemcpyAsync(dst.get(), src.get(), n * 4, hipMemcpyDeviceToDevice, s));
      };
      t->offs = DBuf<int64_t>(pl.n_sub, nullptr);
      GB_HIP(hipMemcpyAsync(t->offs.get(), pl.off.data(), pl.n_sub * 8, hipMemcpyHostToDevice, s));
      t->npad = DBuf<int32_t>(pl.n_sub, nullptr);
      GB_HIP(hipMemcpyAsync(t->npad.get(), npad, pl.n_sub * 4, hipMemcpyDeviceToDevice, s));
      t->tiles = DBuf<int4>(t->pl.launch.size(), nullptr);
      GB_HIP(hipMemcpyAsync(t->tiles.get(), t->pl.launch.data(),
                            t->pl.launch.size() * sizeof(int4), hipMemcpyHostToDevice, s));
      dup_i32(t->core_ptr, P.core_ptr, P.n_sub + 1);
      dup_i32(t->sub_ptr, P.sub_ptr, P.n_sub + 1);
      dup_i32(t->sub_idx, P.sub_idx, P.total);
      dup_i32(t->sub_pos, P.sub_pos, P.total);
      t->ckpt.emplace_back(pl.total * 8, s);
      GB_HIP(hipMemcpyAsync(t->ckpt[0].p, X64, pl.total * 8, hipMemcpyDeviceToDevice, s));
      GB_HIP(hipStreamSynchronize(s));  // host plan vectors above are copied before return
    }
    GB_HIP(hipEventRecord(t_gather.b, s));
  }

  // (with split-bf16 squares tile_policy picks that kernel's variant; the FP64 refinement tunes
  // its own tile edge)
  // (after split squares the plan holds the split's tile edges; FP64 squares on whole blocks --
  // the refinement's fallback, refine_kind 1 and 2 -- tune their own variant when they run)
  auto ensure_xd = [&] {
    if (xd_ready) return;
    hipLaunchKernelGGL((k_convert<float, double>), dim3(grid_for(pl.total, kT, 65536)), dim3(kT),
                       0, s, xs, xd, pl.total, xs_scale);
    GB_LAUNCH_CHECK();
    xd_ready = true;
  };
  auto fp64_tiles_for_blocks = [&] {  // (32-edge tiles take squares only)
    if (low && (planes > 0 || pl.lg.n[variant_index(32)] > 0))
      choose_tiles<double>(P, pl, xd, sd, tiles, offs, s, 5, 0, st, xcd, per_sub, 0, false);
  };
  CoreRows cr;
  const double* rows_final = nullptr;  // core-row refinement: the core rows of D and of D^2
  const double* rows_check = nullptr;
  Timer& t_loop = low ? t_ref : t_sp2;
  GB_HIP(hipEventRecord(t_loop.a, s));
  if (low && done) {
    // converged during the FP64 steps: nothing to refine
  } else if (low && (o.refine_kind == 0 || o.refine_kind == 2)) {
    // FP64 refinement by purification, which drives every eigenvalue to 0 or 1 without acting on
    // the trace, so the occupation the low-precision loop reached is kept.  The stop test takes
    // the traces from X itself, so no square is spent on it.
    // Core rows (refine_kind 0): S_3 .. S_6 of X in turn (see smooth_coef; S_2 first where its
    // 3 e^2 will do, S_2 alone for n_refine = 1) until the stop test holds with two decades to
    // spare, at the last one holds.  If it never does and an eigenvalue too far from 0 and 1 is the
    // cause, the low-precision loop goes on to its rounding floor; whole-block steps follow where
    // that does not help either.
    bool refined = false;
    // Does the low-precision loop go on after a refinement that ended at e?  Not where e is short
    // of idem_tol by rounding only (the default tolerance is met): more low-precision squares would
    // add theirs and resolve nothing.
    auto resumes = [&](double e) { return stop_kind == 5 && e > 1e-10 * N / 1024.0; };
    if (o.refine_kind == 0 && xs && core_rows_plan(P, pl, cr, s)) {
      DBuf<double> part(2 * (size_t)pl.n_sub, s);
      DBuf<RefineState> rs(1, s);
      int32_t* const rdone = &rs.get()->done;
      double* sl = ws->get<double>(7, 5 * (size_t)cr.total, s);
      const RowsCtx rc{cr, pl, P, offs, npad, s, xs_scale};
      auto y_of = [&](int m) { return sl + (2 + m % 3) * cr.total; };  // S_6 follows S_3 in place
      auto check = [&](const double* y, double thr, int m) {
        hipLaunchKernelGGL(k_trace_rows<double>, dim3(pl.n_sub), dim3(kT), 0, s, y,
                           cr.soffs.get(), npad, P.core_ptr.get(), part.get(), rdone, 1.0,
                           1.0);
        hipLaunchKernelGGL(k_refine_check, dim3(1), dim3(kT), 0, s, part.get(), pl.n_sub,
                           (double)n_occ, thr, m, rs.get());
        GB_LAUNCH_CHECK();
      };
      // the terms m .. 2m - 1 of S_m, for the orders lo .. hi, in the product that gives V X^j
      auto terms = [&](int j, int lo, int hi, auto&& slab) {
        RowsAcc a{};
        for (int m = lo; m <= hi; ++m)
          if (m <= j && j < 2 * m) {
            if (m == j) a.fresh |= 1 << a.n;
            a.y[a.n] = slab(m);
            a.c[a.n++] = smooth_coef(m, j);
          }
        return a;
      };
      RefineState h;
      for (int attempt = 0; attempt < 2; ++attempt) {
        const int lo = n_refine == 1 || 3.0 * st.idem * st.idem <= 1e-2 * tol ? 2 : 3;
        // the highest order whose equivalent in McWeeny steps (below) is within the limit given
        const int hi = n_refine == 1 ? 2 : n_refine == 2 ? 4 : n_refine == 3 ? 5 : kSmoothMax;
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(kT), 0, s, rdone, (int64_t)1);
        double *v = sl, *w = sl + cr.total;
        hipLaunchKernelGGL(k_rows_copy<float>, dim3((pl.max_npad + 63) / 64, pl.n_sub), dim3(256),
                           0, s, xs, offs, npad, v, cr.soffs.get(), P.core_ptr.get(),
                           xs_scale);
        GB_LAUNCH_CHECK();
        check(v, tol, 1);
        for (int j = 2; j < 2 * hi; ++j) {
          rc.mm(xs, v, j + 1 < 2 * hi ? w : nullptr, terms(j, lo, hi, y_of), rdone);
          std::swap(v, w);
          const int m = (j + 1) / 2;
          if (j % 2 && m >= lo) check(y_of(m), m == hi ? tol : 1e-2 * tol, m);
        }
        GB_HIP(hipMemcpyAsync(&h, rs.get(), sizeof(h), hipMemcpyDeviceToHost, s));
        GB_HIP(hipStreamSynchronize(s));
        if (h.done || !resumes(h.rec.e)) break;
        run_low(0.0);
      }
      refined = h.done > 0;
      if (refined) {
        const int m = h.done;
        rows_final = m == 1 ? sl : y_of(m);
        if (o.check_idem) {
          // the check's square: Z = Y S_m(X), the core rows of D^2 (2m - 1 more slab products;
          // only when the max-norm check is asked for)
          double* z = y_of(m + 1);
          double *v = sl, *w = sl + cr.total;
          if (m == 1) {
            rc.mm(xs, rows_final, z);
          } else {
            rc.mm(xs, rows_final, v);
            for (int j = 2; j < 2 * m; ++j) {
              rc.mm(xs, v, w, terms(j, m, m, [&](int) { return z; }));
              std::swap(v, w);
            }
          }
          rows_check = z;
        }
        // in McWeeny steps: what 2^steps >= m takes, one more for S_6, which may end at the
        // tolerance itself
        st.n_refine_done = m == 1 ? 0 : m == 2 ? 1 : m <= 4 ? 2 : m - 2;
        const int at = std::min(it_end, 127);
        st.idem = h.rec.e;
        st.t1[at] = h.rec.t1;
        st.t2[at] = h.rec.t2;
        stop_kind = 1;
      }
    }
    if (!refined) {
      // Whole blocks: X^2 = S, then 3S - 2 S X (S and X commute, so S X is computed on upper
      // tiles and mirrored); steps repeat until the FP64 stop test holds (at most n_refine,
      // default 8).  Eight steps do not take an eigenvalue within a tenth of 1/2 to an end (two
      // pairs of sites, of which one reaches a single site of the other): if the loop before them
      // was cut short, it goes on and they start again.
      DBuf<double> part(2 * (size_t)pl.n_sub, s);
      double* td = ws->get<double>(2, pl.total, s);
      const int max_steps = n_refine > 0 ? n_refine : 8;
      StepRec r;
      for (;;) {
        ensure_xd();
        fp64_tiles_for_blocks();
        st.n_refine_done = 0;
        for (int step = 0;; ++step) {
          hipLaunchKernelGGL(k_trace_rows<double>, dim3(pl.n_sub), dim3(kT), 0, s, xd, offs,
                             npad, P.core_ptr.get(), part.get(), nullptr, 1.0, 1.0);
          hipLaunchKernelGGL(k_decide, dim3(1), dim3(kT), 0, s, part.get(), pl.n_sub,
                             (double)n_occ, tol, 2, 0, recs.get());
          GB_LAUNCH_CHECK();
          GB_HIP(hipMemcpyAsync(&r, recs.get(), sizeof(r), hipMemcpyDeviceToHost, s));
          GB_HIP(hipStreamSynchronize(s));
          if (r.e <= tol || step == max_steps) break;
          launch_square<double>(xd, sd, tiles.get(), pl.lg, offs, s);
          launch_symm<double, 1>(sd, xd, sd, td, -2.0, 3.0, tiles.get(), pl.lg, offs, s);
          std::swap(xd, td);
          ++st.n_refine_done;
        }
        if (r.e <= tol || !resumes(r.e)) break;
        run_low(0.0);
      }
      const int at = std::min(it_end, 127);
      st.idem = r.e;
      st.t1[at] = r.t1;
      st.t2[at] = r.t2;
      stop_kind = r.e <= tol ? 1 : 2;
    }
  } else if (low) {
    // FP64 refinement: SP2 steps with FP64 traces from where the FP32 loop stopped
    ensure_xd();
    fp64_tiles_for_blocks();
    const uint8_t* bin = nullptr;
    int nbin = 0;
    if (o.branch_in && o.n_branch_in > it_end) {
      bin = o.branch_in;
      nbin = o.n_branch_in;
    }
    // Without a replayed sequence the steps alternate X^2 and 2X - X^2 (the first one chosen
    // by the trace rule): each pair squares the distance of every eigenvalue from 0 or 1, as a
    // McWeeny step does, and leaves the trace where the low-precision loop put it.  The trace
    // rule itself would steer towards n_occ, which the rounded partitioned trace cannot reach
    // with idempotent blocks, and cycles.
    const int cap = std::min(it_end + (n_refine > 0 ? n_refine : 16), 127);
    it_end = sp2_loop<double>(xd, sd, pl, tiles, offs, npad, P, n_occ, tol, cap, bin, nbin, false,
                              it_end, st, recs, s, &stop_kind, nullptr, 0, per_sub,
                              bin == nullptr);
  } else {
    if (dev_loop && !tape_out)
      it_end = sp2_loop_dev<double>(xd, sd, pl, tiles, offs, npad, P, n_occ, tol, max_iter,
                                    o.branch_in, o.n_branch_in, false, 0, st, s, &stop_kind, 0,
                                    o.launch_mode == 2);
    else
      it_end = sp2_loop<double>(xd, sd, pl, tiles, offs, npad, P, n_occ, tol, max_iter,
                                o.branch_in, o.n_branch_in, false, 0, st, recs, s, &stop_kind,
                                tape_out ? *tape_out : nullptr, 0, per_sub);
    if (tape_out) (*tape_out)->K = it_end;
  }
  GB_HIP(hipEventRecord(t_loop.b, s));
  st.iters = it_end;
  st.converged = stop_kind == 1 ? 1 : 0;

  // final idempotency check on the core rows: X^2 restricted to the tiles that hold them (all
  // upper tiles in tile rows below the core size), then max |X^2 - X| over the core rows
  // (after the core-row refinement the core rows of X and X^2 are already there)
  // (only with check_idem: the trace-based FP64 stop test above is the default check)
  if (!rows_final) ensure_xd();
  const double* xfin = rows_final ? rows_final : xd;
  const int64_t* foffs = rows_final ? cr.soffs.get() : offs;
  DBuf<int4> idem_tiles;
  DBuf<double> per, mx;
  if (o.check_idem) {
    if (!rows_final) {
      idem_tiles = DBuf<int4>(std::max<size_t>(pl.idem.size(), 1), s);
      GB_HIP(hipMemcpyAsync(idem_tiles.get(), pl.idem.data(), pl.idem.size() * sizeof(int4),
                            hipMemcpyHostToDevice, s));
      launch_square<double>(xd, sd, idem_tiles.get(), one_group(128, (int)pl.idem.size()),
                            offs, s);
    }
    const double* sfin = rows_final ? rows_check : sd;
    per = DBuf<double>(pl.n_sub, s);
    mx = DBuf<double>(1, s);
    hipLaunchKernelGGL(k_idem<double>, dim3(pl.n_sub), dim3(kT), 0, s, xfin, sfin, foffs,
                       npad, P.core_ptr.get(), P.sub_ptr.get(), per.get());
    GB_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_max, dim3(1), dim3(kT), 0, s, per.get(), pl.n_sub, mx.get());
    GB_LAUNCH_CHECK();
  }
  // scatter
  GB_HIP(hipEventRecord(t_scat.a, s));
  hipLaunchKernelGGL(k_scatter<double>, dim3(N), dim3(kT), 0, s, xfin, foffs, npad,
                     P.sub_ptr.get(), P.sub_idx.get(), P.sub_pos.get(), P.col_sub.get(),
                     P.col_loc.get(), D.width, D.col, D.val);
  GB_LAUNCH_CHECK();
  GB_HIP(hipEventRecord(t_scat.b, s));
  double idem_max = NAN;
  if (o.check_idem) GB_HIP(hipMemcpyAsync(&idem_max, mx.get(), 8, hipMemcpyDeviceToHost, s));
  GB_HIP(hipEventRecord(t_all.b, s));
  GB_HIP(hipStreamSynchronize(s));
  st.ms_gather = elapsed(t_gather.a, t_gather.b);
  st.ms_sp2 = elapsed(t_sp2.a, t_sp2.b);
  if (low) st.ms_refine = elapsed(t_ref.a, t_ref.b);
  st.ms_scatter = elapsed(t_scat.a, t_scat.b);
  st.idem_max = idem_max;
  const int last = std::min(it_end, 127);
  st.trace = st.t1[last];
  st.ms_total += elapsed(t_all.a, t_all.b);
}


void tape_destroy(TapeData* t) { delete t; }
void tape_dims(const TapeData* t, int* n, int* max_sub) {
  *n = t->N;
  *max_sub = t->max_sub;
}

// Reverse sweep: Gbar <- Gbar X + X Gbar (X <- X^2) or 2 Gbar - (Gbar X + X Gbar)
// (X <- 2X - X^2) from the last step to the first, recomputing each checkpoint segment
// forward; then dL/dH per slot of H.
void density_vjp(TapeData& t, const gb_ell& G_D, const gb_ell& H, double* G_H, hipStream_t s) {
  const Plan& pl = t.pl;
  const int K = t.K, c = t.stride;
  WsLease ws;  // the batch buffers of the expansions: Gbar, its successor, a segment's iterates
  double* G = ws->get<double>(0, pl.total, s);
  double* G2 = ws->get<double>(1, pl.total, s);
  double* const seg = c > 1 ? ws->get<double>(5, (c - 1) * (size_t)pl.total, s) : nullptr;
  const int gfill = grid_for(pl.total, kT, 65536);
  hipLaunchKernelGGL(k_fill, dim3(gfill), dim3(kT), 0, s, G, pl.total, 0.0);
  GB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_seed, dim3(pl.n_sub), dim3(kT), 0, s, G_D.val, G_D.width, t.core_ptr.get(),
                     t.sub_ptr.get(), t.sub_idx.get(), t.sub_pos.get(), t.offs.get(), t.npad.get(),
                     G);
  GB_LAUNCH_CHECK();
  for (int m = (K - 1) / c; m >= 0 && K > 0; --m) {
    const int start = m * c, end = std::min(start + c, K);
    std::vector<double*> xs;
    xs.push_back(static_cast<double*>(t.ckpt[m].p));
    for (int n = start; n + 1 < end; ++n) {
      double* xin = xs.back();
      double* xout = seg + (int64_t)(n - start) * pl.total;
      launch_plan_square_f64(xin, xout, pl, t.tiles.get(), t.offs.get(), s, t.branch[n] == 1);
      xs.push_back(xout);
    }
    for (int n = end - 1; n >= start; --n) {
      const double* X = xs[n - start];
      const double c1 = t.branch[n] == 0 ? 1.0 : -1.0, c2 = t.branch[n] == 0 ? 0.0 : 2.0;
      // the seed holds core rows and columns only
      const int klim = n == K - 1 ? t.max_core : 0;
      hipLaunchKernelGGL((k_symm_mm<double, 2, 64, 2, 1>), dim3(pl.lg.n[variant_index(62)]),
                         dim3(kT), 0, s, G, X, G, G2, c1, c2, t.tiles.get(),
                         t.offs.get(), (const int32_t*)nullptr, 0, (const int32_t*)nullptr, klim);
      GB_LAUNCH_CHECK();
      std::swap(G, G2);
    }
  }
  // vertex -> subgraph index and the deterministic assembly on H's pattern
  const int n = t.N;
  DBuf<int32_t> cnt(n, s), fill(n, s), vs_ptr(n + 1, s);
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kT)), dim3(kT), 0, s, cnt.get(), (int64_t)n);
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kT)), dim3(kT), 0, s, fill.get(), (int64_t)n);
  GB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_vs_count, dim3(pl.n_sub), dim3(kT), 0, s, t.sub_ptr.get(), t.sub_idx.get(),
                     cnt.get());
  GB_LAUNCH_CHECK();
  exclusive_scan_i32(cnt.get(), vs_ptr.get(), n, s);
  int32_t tot = 0;
  GB_HIP(hipMemcpyAsync(&tot, vs_ptr.get() + n, 4, hipMemcpyDeviceToHost, s));
  GB_HIP(hipStreamSynchronize(s));
  DBuf<int32_t> raw_sub(tot, s), raw_loc(tot, s), vs_sub(tot, s), vs_loc(tot, s);
  hipLaunchKernelGGL(k_vs_fill, dim3(pl.n_sub), dim3(kT), 0, s, t.sub_ptr.get(), t.sub_idx.get(),
                     vs_ptr.get(), fill.get(), raw_sub.get(), raw_loc.get());
  GB_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_vs_sort, dim3((n + kT / 64 - 1) / (kT / 64)), dim3(kT), 0, s, n,
                     vs_ptr.get(), raw_sub.get(), raw_loc.get(), vs_sub.get(), vs_loc.get());
  GB_LAUNCH_CHECK();
  const int64_t slots = (int64_t)H.n * H.width;
  hipLaunchKernelGGL(k_assemble, dim3(grid_for(slots, kT)), dim3(kT), 0, s, H.col, H.n, H.width,
                     vs_ptr.get(), vs_sub.get(), vs_loc.get(), t.offs.get(), t.npad.get(), G,
                     -1.0 / (t.emax - t.emin), G_H);
  GB_LAUNCH_CHECK();
  GB_HIP(hipStreamSynchronize(s));
}


// ---- finite-temperature Fermi-operator expansion (Eq. 7; terms by the recurrence of Eq. 5,
// per subgraph as in Eq. 6) ----------------------------------------------------------------

namespace {

// The expansion needs only the core rows of T_n(Ht): with V_n = E T_n for the core unit rows E,
// V_{n+1} = 2 V_n Ht - V_{n-1}, one row never reads another one, and Ht is as sparse as H.  So a
// workgroup carries R core rows of one subgraph through the whole recurrence with V_n and V_{n-1}
// in LDS, and the only traffic of a term is Ht's entries on the subgraph.
//
// Those entries, per subgraph, for pairs of neighbouring columns 2p and 2p + 1 (two orbitals of a
// site, as a rule, which couple to the same others): slot t of pair p at eoff[s] + t npad / 2 + p
// (a wave of consecutive pairs reads consecutive words) holds the local index of the other end as
// 16 bits (a subgraph is limited to about 13600 vertices by the gather's LDS) and both values of
// Ht = (2h - (e_max + e_min) delta) / (e_max - e_min), zero where a column has no such entry;
// len counts a pair's slots, in whole groups of kFoePad, the last one filled with zeros.
//
// Which slot an entry takes decides the bank conflicts of the recurrence: LDS serves a 16-byte
// read sixteen lanes at a time from sixteen banks, and slot q of sixteen pairs names sixteen
// scattered columns, 2.6 clocks' worth where one would do.  So the r-th entry of each residue c mod
// 16 takes slot 16 r + (c - g) mod 16, g being the pair's rank among the sixteen: slot q then reads
// bank q + g.  Entries past the end fill the holes that short residues leave (conflicts down by
// three quarters; N = 1024 4.51 -> 4.11 ms of recurrence for 0.13 ms of sorting).
// A wave per pair, lanes side by side in a row of H (a thread per column took 0.39 ms; now 0.29
// with the order, 0.16 without).
constexpr int kFoePad = 8;
__device__ inline int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
// Rank of a lane among the sixteen that a 16-byte LDS read serves together (lanes 0-3, 12-15,
// 20-23, 24-27, then 4-7, 8-11, 16-19, 28-31, and the same of the upper half).
__device__ __forceinline__ int lds_rank(int lane) { return (lane & 31) / 8 * 4 + (lane & 3); }
constexpr int kPairsPerBlock = 16;
__global__ __launch_bounds__(kT) void k_foe_ell(const int32_t* __restrict__ hcol,
                                                const double* __restrict__ hval, int w, double emin,
                                                double emax, const int32_t* __restrict__ core_ptr,
                                                const int32_t* __restrict__ sub_ptr,
                                                const int32_t* __restrict__ sub_idx,
                                                const int64_t* __restrict__ eoff,
                                                const int32_t* __restrict__ npad,
                                                uint16_t* __restrict__ idx,
                                                double* __restrict__ val,
                                                int32_t* __restrict__ len, int ordered) {
  extern __shared__ __align__(16) unsigned char smem[];
  int32_t* sub = reinterpret_cast<int32_t*>(smem);
  const int s = blockIdx.x;
  const int b = sub_ptr[s], n = sub_ptr[s + 1] - b, n2 = (n + 1) / 2;
  if ((int)blockIdx.y * kPairsPerBlock >= n2) return;  // the whole workgroup leaves together
  const int k = core_ptr[s + 1] - core_ptr[s], hp = npad[s] / 2;
  for (int a = threadIdx.x; a < n; a += blockDim.x) sub[a] = sub_idx[b + a];
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  // per wave: pos[n]; where the order is chosen, cl[2w] (local indices, then slots), hl[2w], ul[2w]
  const int cap = ordered ? 2 * w : 0;
  uint16_t* pos = reinterpret_cast<uint16_t*>(sub + n) + (int64_t)wave * (n + 2 * cap + (cap + 1) / 2);
  uint16_t *cl = pos + n, *hl = cl + cap;
  uint8_t* ul = reinterpret_cast<uint8_t*>(hl + cap);
  const uint64_t below = (1ull << lane) - 1;
  // local index of vertex j: in the core run [0, k) or the halo run [k, n), both ascending; or -1
  auto local = [&](int32_t j) {
    int lo = 0, hi = k;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sub[mid] < j) lo = mid + 1;
      else hi = mid;
    }
    if (lo < k && sub[lo] == j) return lo;
    lo = k;
    hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sub[mid] < j) lo = mid + 1;
      else hi = mid;
    }
    return lo < n && sub[lo] == j ? lo : -1;
  };
  const int end = min(n2, ((int)blockIdx.y + 1) * kPairsPerBlock);
  for (int p = blockIdx.y * kPairsPerBlock + wave; p < end; p += waves) {
    uint16_t* ip = idx + eoff[s] + p;
    double* vp = val + 2 * (eoff[s] + p);
    for (int a = lane; a < n; a += 64) pos[a] = 0xffff;
    __threadfence_block();
    // the pair's list: what column 2p couples to, then what only 2p + 1 does
    int m = 0;
    for (int x = 0; x < 2 && 2 * p + x < n; ++x) {
      const int i = sub[2 * p + x];
      for (int t0 = 0; t0 < w; t0 += 64) {
        const int t = t0 + lane;
        const int32_t j = t < w ? hcol[(int64_t)i * w + t] : -1;
        const int loc = j < 0 ? -1 : local(j);
        const bool fresh = loc >= 0 && (x == 0 || pos[loc] == 0xffff);
        const uint64_t mask = __ballot(fresh);
        if (fresh) {
          const int q = m + __popcll(mask & below);
          pos[loc] = (uint16_t)q;
          if (ordered) cl[q] = (uint16_t)loc;
        }
        m += __popcll(mask);
      }
      __threadfence_block();
    }
    if (ordered) {
      // slot 16 r + (c - g) mod 16 for the r-th entry of residue c mod 16, where that is below m;
      // the others fill the holes
      const int g = lds_rank(p & 63);
      int count = 0;  // of residue `lane`
      for (int q0 = 0; q0 < m; q0 += 64) {
        const int q = q0 + lane, c = q < m ? cl[q] & 15 : -1;
        int r = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const uint64_t mask = __ballot(c == e);
          const int had = lane_value(count, e);
          if (c == e) r = had + __popcll(mask & below);
          if (lane == e) count += __popcll(mask);
        }
        if (q < m) cl[q] = (uint16_t)(16 * r + ((c - g) & 15));
      }
      for (int t = lane; t < m; t += 64) ul[t] = 0;
      __threadfence_block();
      for (int q = lane; q < m; q += 64)
        if (cl[q] < m) ul[cl[q]] = 1;
      __threadfence_block();
      int holes = 0;
      for (int t0 = 0; t0 < m; t0 += 64) {
        const bool hole = t0 + lane < m && !ul[t0 + lane];
        const uint64_t mask = __ballot(hole);
        if (hole) hl[holes + __popcll(mask & below)] = (uint16_t)(t0 + lane);
        holes += __popcll(mask);
      }
      __threadfence_block();
      int out = 0;
      for (int q0 = 0; q0 < m; q0 += 64) {
        const bool late = q0 + lane < m && cl[q0 + lane] >= m;
        const uint64_t mask = __ballot(late);
        if (late) cl[q0 + lane] = hl[out + __popcll(mask & below)];
        out += __popcll(mask);
      }
      __threadfence_block();
    }
    // both columns' values over zeros, which also fill the last group
    const int full = (m + kFoePad - 1) / kFoePad * kFoePad;
    for (int t = lane; t < full; t += 64) {
      ip[(int64_t)t * hp] = 0;
      vp[2 * (int64_t)t * hp] = vp[2 * (int64_t)t * hp + 1] = 0.0;
    }
    if (lane == 0) len[b + p] = full;
    __threadfence_block();
    for (int x = 0; x < 2 && 2 * p + x < n; ++x) {
      const int i = sub[2 * p + x];
      for (int t0 = 0; t0 < w; t0 += 64) {
        const int t = t0 + lane;
        const int32_t j = t < w ? hcol[(int64_t)i * w + t] : -1;
        const int loc = j < 0 ? -1 : local(j);
        if (loc < 0) continue;
        const int q = ordered ? cl[pos[loc]] : pos[loc];
        const double h =
            (2.0 * hval[(int64_t)i * w + t] - (j == i ? emax + emin : 0.0)) / (emax - emin);
        ip[(int64_t)q * hp] = (uint16_t)loc;
        vp[2 * (int64_t)q * hp + x] = h;
      }
    }
  }
}

// The recurrence of R core rows r0 .. r0 + R - 1 of one subgraph up to V_nterm (rows beyond the
// core are zero rows).  LDS: V_n and V_{n-1}, columns side by side in pairs of rows (one 16-byte
// read per pair), V_{n+1} overwriting V_{n-1} entry by entry; one barrier per term.  SPILL: a
// subgraph too large for two LDS arrays keeps V_{n-1} in global memory and swaps after each term.
//   coef: dacc (core-row slabs at soffs, row stride npad) = sum_n coef[n] V_n.
//   hist: with coef NULL, V_{n+1} of every product is kept there (slabs as dacc's, hist_ld apart);
//         with coef and t_from > 0 the terms up to t_from are read from it and the recurrence
//         goes on from there (order 160 with mu solved: 160 products, not 240; N = 1024, 0.6 GB
//         kept, 12.0 -> 8.1 ms).
//   part: for the first ntr products n -> n + 1, sum V_n V_{n+1} and sum V_{n+1}^2 over the rows:
//         T_m T_n = (T_{m+n} + T_{|m-n|}) / 2 turns them into the core traces t_{2n+1} and
//         t_{2n+2}, so the traces of M terms take M / 2 products.
// An entry of Ht reads R doubles of V_n in LDS at a scattered column, which bounded the recurrence
// with a thread per column (LDS active 72 % of the time, mostly bank conflicts).  So a thread takes
// two columns that couple to the same others, which halves the reads, the lists are ordered by bank
// (above), and R = 4 rows share an entry: eight products for two reads and 18 bytes of Ht.  What
// bounds it now is those bytes out of L2: with half the rows per workgroup, twice the bytes, the
// recurrence takes 6.45 ms for 4.11.  Lists are whole groups of U slots, a slot's address the
// wave's plus the lane's pair: a test per slot cost more instructions than the products (5.35
// against 4.77 ms).  Order 160 at N = 1024 (64 subgraphs of ~900; whole call) 8.1 -> 4.8 ms against
// a column per thread, 26 us per term (as full products of whole blocks, each term 2 n^3 flops and
// five passes over the batch, 2.2 ms); N = 18000 (565 subgraphs of ~1200) 140 -> 84 ms, 0.50 ms per
// term (57.6).  U = 4 5.0, U = 16 4.9 ms; workgroups of at most 512 threads: N = 18000 105 ms.
template <int R, bool SPILL>
__global__ __launch_bounds__(1024) void k_foe_rows(
    const int4* __restrict__ items, const uint16_t* __restrict__ idx,
    const double* __restrict__ val, const int32_t* __restrict__ len,
    const int64_t* __restrict__ eoff, const int32_t* __restrict__ sub_ptr,
    const int32_t* __restrict__ core_ptr, const int64_t* __restrict__ soffs, int nterm, int ntr,
    const double* __restrict__ coef, double* __restrict__ dacc, double* __restrict__ part,
    double* __restrict__ spill, int spill_ld, double* __restrict__ hist, int64_t hist_ld,
    int t_from) {
  constexpr int E = R >= 2 ? 2 : 1, PL = R / E, U = kFoePad;
  static_assert(!SPILL || R == 1, "the spilled form carries one row");
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[2][2][16];
  double* mine = part ? part + (int64_t)blockIdx.x * 2 * ntr : nullptr;
  const int4 it = items[blockIdx.x];
  if (it.x < 0) {  // padding entry of an XCD queue
    for (int q = threadIdx.x; q < 2 * ntr; q += blockDim.x) mine[q] = 0.0;
    return;
  }
  const int s = it.x, r0 = it.y, np = it.w;
  const int b = sub_ptr[s], n = sub_ptr[s + 1] - b;
  const int kr = min(R, core_ptr[s + 1] - core_ptr[s] - r0);
  double* cur = reinterpret_cast<double*>(smem);
  double* prev = SPILL ? spill + (int64_t)blockIdx.x * spill_ld : cur + R * n;
  const uint16_t* ix = idx + eoff[s];
  const double* hv = val + 2 * eoff[s];
  const int hp = np / 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  const int64_t slab = soffs[s] + (int64_t)r0 * np;
  for (int a = threadIdx.x; a < n; a += blockDim.x)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double v = r < kr && a == r0 + r ? 1.0 : 0.0, u = 0.0;
      if (t_from > 0 && r < kr) {  // V_{t_from}, V_{t_from - 1}; the terms so far in their order
        const double* hr = hist + slab + (int64_t)r * np + a;
        double d = coef[0] * v;
        for (int m = 1; m <= t_from; ++m) {
          u = v;
          v = hr[(m - 1) * hist_ld];
          d += coef[m] * v;
        }
        dacc[slab + (int64_t)r * np + a] = d;
      }
      cur[((r / E) * n + a) * E + r % E] = v;
      prev[((r / E) * n + a) * E + r % E] = u;
    }
  __syncthreads();
  for (int t = t_from; t < nterm; ++t) {
    double p0 = 0.0, p1 = 0.0;
    for (int p2 = threadIdx.x; 2 * p2 < n; p2 += blockDim.x) {
      double acc[2][R];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[0][r] = acc[1][r] = 0.0;
      const int L = len[b + p2];
      for (int q = 0; q < L; q += U) {
        double h[U][2];
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // the slot's row is the wave's, the pair the lane's
          const int64_t row = (int64_t)(q + u) * hp;
          c[u] = (ix + row)[p2];
          __builtin_memcpy(h[u], __builtin_assume_aligned(hv + 2 * row + 2 * p2, 16), 16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int p = 0; p < PL; ++p) {
            double v[E];
            __builtin_memcpy(v, __builtin_assume_aligned(cur + (p * n + c[u]) * E, 8 * E), 8 * E);
#pragma unroll
            for (int x = 0; x < E; ++x) {
              acc[0][p * E + x] = __builtin_fma(v[x], h[u][0], acc[0][p * E + x]);
              acc[1][p * E + x] = __builtin_fma(v[x], h[u][1], acc[1][p * E + x]);
            }
          }
      }
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const int a = 2 * p2 + y;
        if (a >= n) break;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int o = ((r / E) * n + a) * E + r % E;
          const double v = cur[o];
          const double nv = t == 0 ? acc[y][r] : 2.0 * acc[y][r] - prev[o];
          prev[o] = nv;
          p0 += v * nv;
          p1 += nv * nv;
          if (coef && r < kr) {
            double* d = dacc + slab + (int64_t)r * np + a;
            *d = t == 0 ? coef[0] * v + coef[1] * nv : *d + coef[t + 1] * nv;
          } else if (hist && r < kr) {
            hist[t * hist_ld + slab + (int64_t)r * np + a] = nv;
          }
        }
      }
    }
    if (t < ntr) {
      for (int o = 32; o > 0; o >>= 1) {
        p0 += __shfl_xor(p0, o);
        p1 += __shfl_xor(p1, o);
      }
      if (lane == 0) {
        red[t & 1][0][wave] = p0;
        red[t & 1][1][wave] = p1;
      }
    }
    __syncthreads();
    if (t < ntr && threadIdx.x < 2) {
      double v = 0.0;
      for (int q = 0; q < nwave; ++q) v += red[t & 1][threadIdx.x][q];
      mine[2 * t + threadIdx.x] = v;
    }
    if (SPILL) {
      for (int a = threadIdx.x; a < n; a += blockDim.x) {
        const double v = cur[a];
        cur[a] = prev[a];
        prev[a] = v;
      }
      __syncthreads();
    } else {
      double* x = cur;
      cur = prev;
      prev = x;
    }
  }
}

// out[q] = the sum over the workgroups of k_foe_rows of part[.][q] (one workgroup per q)
__global__ __launch_bounds__(kT) void k_foe_sums(const double* __restrict__ part, int n_items,
                                                 int nq, double* __restrict__ out) {
  __shared__ double red[kT];
  const int q = blockIdx.x;
  double v = 0.0;
  for (int i = threadIdx.x; i < n_items; i += kT) v += part[(int64_t)i * nq + q];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[q] = red[0];
}

// ---- Fermi function coefficients and mu on the device ----------------------------------------
// What chebyshev_fermi and foe_solve_mu below compute on the host, from the traces to the
// coefficients, next to the recurrence: 2 (M + 1) K cosines and some 55 K exponentials (M = 160, K
// = 1024) kept the host busy for 3 of the call's 15.0 ms while the device waited (now 12.0 ms).
// The arguments are rounded as the host's are, n times theta_k.
__device__ double node_theta(int k, int K) { return M_PI * (k + 0.5) / K; }

// energies and weights of the nodes: sum_n c_n(mu) t_n = sum_k f(e_k; mu) w_k (wave per node)
__global__ __launch_bounds__(kT) void k_foe_nodes(const double* __restrict__ traces, int M, int K,
                                                  double mid, double half, double* __restrict__ e,
                                                  double* __restrict__ w) {
  const int k = blockIdx.x * (kT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (k >= K) return;
  const double th = node_theta(k, K);
  double acc = lane == 0 ? 0.5 * traces[0] : 0.0;
  for (int n = 1 + lane; n <= M; n += 64) acc += cos(n * th) * traces[n];
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane == 0) {
    e[k] = mid + half * cos(th);
    w[k] = acc * (2.0 / K);
  }
}

__device__ double fermi_dev(double e, double beta, double mu) {
  return 1.0 / (1.0 + exp(beta * (e - mu)));
}

// mu with sum_k f(e_k; mu) w_k = n_occ by halving [emin, emax], as on the host (the sum of a
// truncated expansion may cross n_occ more than once): out = {mu, the sums at emin and emax}.
// Fifteen waves take the fifteen midpoints that four halvings can ask for, so 14 rounds do for 55.
__global__ __launch_bounds__(960) void k_foe_mu(const double* __restrict__ e,
                                                const double* __restrict__ w, int K, double emin,
                                                double emax, double beta, double n_occ,
                                                double* __restrict__ out) {
  __shared__ double sum[16];
  const int node = 1 + (threadIdx.x >> 6), lane = threadIdx.x & 63;  // root 1, below, above: 2q, 2q + 1
  auto occupation = [&](double mu) {
    double t = 0.0;
    for (int k = lane; k < K; k += 64) t += fermi_dev(e[k], beta, mu) * w[k];
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    return t;
  };
  double lo = emin, hi = emax;
  if (node <= 2) {
    const double t = occupation(node == 1 ? emin : emax);
    if (lane == 0) out[node] = t;
  }
  bool open = true;
  for (int it = 0; it < 400 && open; it += 4) {  // every thread holds the same lo and hi
    double a = lo, b = hi, x = 0.5 * (lo + hi);
    for (int bit = 30 - __builtin_clz(node); bit >= 0; --bit) {
      if (node >> bit & 1) a = x;
      else b = x;
      x = 0.5 * (a + b);
    }
    const double t = occupation(x);
    if (lane == 0) sum[node] = t - n_occ;
    __syncthreads();
    for (int q = 1, step = 0; step < 4; ++step) {
      const double m = 0.5 * (lo + hi);
      if (!(m > lo && m < hi)) {
        open = false;
        break;
      }
      const bool above = sum[q] < 0.0;
      if (above) lo = m;
      else hi = m;
      q = 2 * q + above;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = 0.5 * (lo + hi);
}

// c[n] = (2/K) sum_k cos(n theta_k) f(e_k; mu), n = 0 halved (one workgroup per n)
__global__ __launch_bounds__(kT) void k_foe_coef(int K, double mid, double half, double beta,
                                                 double mu, double* __restrict__ c) {
  __shared__ double red[kT];
  const int n = blockIdx.x;
  double acc = 0.0;
  for (int k = threadIdx.x; k < K; k += kT) {
    const double th = node_theta(k, K);
    acc += cos(n * th) * fermi_dev(mid + half * cos(th), beta, mu);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) c[n] = red[0] * (2.0 / K) * (n == 0 ? 0.5 : 1.0);
}

int quad_nodes(int order, int n_nodes) { return n_nodes > 0 ? n_nodes : std::max(4 * (order + 1), 1024); }

[[noreturn]] void fail_occupation(double n_occ, double lo, double hi) {
  fail(GB_EINVAL, "n_occ = %g is outside the occupations [%g, %g] reachable in [e_min, e_max]",
       n_occ, lo, hi);
}

double fermi(double e, double beta, double mu) { return 1.0 / (1.0 + std::exp(beta * (e - mu))); }

}  // namespace

void chebyshev_fermi(double emin, double emax, double beta, double mu, int order, int n_nodes,
                     double* c) {
  const int K = quad_nodes(order, n_nodes);
  const double mid = 0.5 * (emax + emin), half = 0.5 * (emax - emin);
  std::vector<double> th(K), f(K);
  for (int k = 0; k < K; ++k) {
    th[k] = M_PI * (k + 0.5) / K;
    f[k] = fermi(mid + half * std::cos(th[k]), beta, mu);
  }
  for (int n = 0; n <= order; ++n) {
    double acc = 0.0;
    for (int k = 0; k < K; ++k) acc += std::cos(n * th[k]) * f[k];
    c[n] = acc * (2.0 / K) * (n == 0 ? 0.5 : 1.0);
  }
}

// sum_n c_n(mu) t_n = sum_k f(e_k; mu) w_k with w_k = (2/K) sum_n' t_n cos(n theta_k) (the n = 0
// term halved): the weights are formed once and each bisection step costs K exponentials.
double foe_solve_mu(const double* traces, int order, double emin, double emax, double beta,
                    double n_occ, int n_nodes) {
  const int K = quad_nodes(order, n_nodes);
  const double mid = 0.5 * (emax + emin), half = 0.5 * (emax - emin);
  std::vector<double> e(K), w(K);
  for (int k = 0; k < K; ++k) {
    const double th = M_PI * (k + 0.5) / K;
    e[k] = mid + half * std::cos(th);
    double acc = 0.5 * traces[0];
    for (int n = 1; n <= order; ++n) acc += std::cos(n * th) * traces[n];
    w[k] = acc * (2.0 / K);
  }
  auto excess = [&](double mu) {
    double t = 0.0;
    for (int k = 0; k < K; ++k) t += fermi(e[k], beta, mu) * w[k];
    return t - n_occ;
  };
  double lo = emin, hi = emax;
  const double glo = excess(lo), ghi = excess(hi);
  if (glo > 0.0 || ghi < 0.0)
    fail_occupation(n_occ, glo + n_occ, ghi + n_occ);
  for (int it = 0; it < 400; ++it) {
    const double m = 0.5 * (lo + hi);
    if (!(m > lo && m < hi)) break;
    if (excess(m) < 0.0) lo = m;
    else hi = m;
  }
  return 0.5 * (lo + hi);
}

// Most memory for the terms that the pass for mu leaves to the pass for D (13 GiB at N = 18000,
// order 160): what a card of 288 GB spares beside a batch.
constexpr size_t kHistMost = (size_t)32 << 30;

void foe(const gb_ell& H, int32_t n_occ, const gb_foe_opts& o, const Part& P, double emin,
         double emax, gb_ell& D, gb_foe_stats& st, hipStream_t s) {
  Timer t_all, t_stage;
  GB_HIP(hipEventRecord(t_all.a, s));
  const int N = H.n, M = o.order, w = H.width;
  // padded sizes, offsets of the subgraphs' entries and of their core-row slabs
  std::vector<int32_t> np(P.n_sub);
  std::vector<int64_t> eo(P.n_sub), so(P.n_sub);
  std::vector<int> order(P.n_sub);
  const int slots = (2 * w + kFoePad - 1) / kFoePad * kFoePad;  // of a pair, at most
  int64_t te = 0, ts = 0;
  int max_np = 0;
  double t0 = 0;  // t_0 = sum of the core sizes
  for (int q = 0; q < P.n_sub; ++q) {
    const int n = P.h_sub_ptr[q + 1] - P.h_sub_ptr[q], k = P.h_core_ptr[q + 1] - P.h_core_ptr[q];
    np[q] = (n + 63) / 64 * 64;
    max_np = std::max(max_np, np[q]);
    eo[q] = te;
    so[q] = ts;
    te += (int64_t)(np[q] / 2) * slots;
    ts += (int64_t)np[q] * k;
    t0 += k;
    order[q] = q;
    st.product_flops += 2.0 * (double)n * n * n;
  }
  if ((size_t)max_np * 8 + (size_t)P.max_sub * 4 + 64 > 160 * 1024)
    fail(GB_EUNSUPPORTED, "subgraph of %d vertices too large", P.max_sub);
  // rows per workgroup: as many as the LDS of one CU holds (see k_foe_rows), at most four; past
  // 10112 vertices not even one row's two arrays fit, and V_{n-1} goes to global memory.  Fewer
  // rows while that leaves at most a workgroup per compute unit (N = 512, 128 groups of four rows:
  // 2.99 -> 2.53 ms with two; N = 1024, 256 groups of four: 4.75 ms, with two 7.1)
  const size_t lds_max = 158 * 1024;
  auto lds_of = [&](int r) { return (size_t)2 * r * P.max_sub * 8; };
  int R = lds_of(4) <= lds_max ? 4 : lds_of(2) <= lds_max ? 2 : 1;
  auto groups = [&](int r) {
    int64_t g = 0;
    for (int q = 0; q < P.n_sub; ++q) g += (P.h_core_ptr[q + 1] - P.h_core_ptr[q] + r - 1) / r;
    return g;
  };
  while (R > 1 && groups(R / 2) <= 256) R /= 2;
  const bool spill = lds_of(1) > lds_max;
  // workgroups per subgraph, largest subgraphs first, each subgraph's on one XCD (its entries of
  // Ht, ~2 MB at n ~ 1000, are read by all of them every term)
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return np[x] > np[y]; });
  std::vector<int4> list, ranges, items;
  for (int q : order) {
    const int k = P.h_core_ptr[q + 1] - P.h_core_ptr[q], first = (int)list.size();
    for (int r = 0; r < k; r += R) list.push_back(make_int4(q, r, 0, np[q]));
    if (k > 0) ranges.push_back(make_int4(first, (int)list.size() - first, 0, q));
  }
  if (o.tile_order == 0) xcd_order(items, list, ranges, 0, ranges.size());
  else items = list;
  const int n_items = (int)items.size();
  DBuf<int32_t> npad(P.n_sub, s), len(P.total, s);
  DBuf<int64_t> eoff(P.n_sub, s), soff(P.n_sub, s);
  DBuf<int4> ditems(n_items, s);
  GB_HIP(hipMemcpyAsync(npad.get(), np.data(), P.n_sub * 4, hipMemcpyHostToDevice, s));
  GB_HIP(hipMemcpyAsync(eoff.get(), eo.data(), P.n_sub * 8, hipMemcpyHostToDevice, s));
  GB_HIP(hipMemcpyAsync(soff.get(), so.data(), P.n_sub * 8, hipMemcpyHostToDevice, s));
  GB_HIP(hipMemcpyAsync(ditems.get(), items.data(), n_items * sizeof(int4),
                        hipMemcpyHostToDevice, s));

  GB_HIP(hipEventRecord(t_stage.a, s));
  WsLease ws;  // cached buffers: Ht's entries on the subgraphs, the core rows of D
  double* const val = ws->get<double>(0, 2 * te, s);
  uint16_t* const idx = ws->get<uint16_t>(1, te, s);
  double* const Dacc = ws->get<double>(2, ts, s);
  // the kernel's LDS: the subgraph, and per wave the slots of its vertices and, where there is
  // room for them, the lists that choose the order
  auto lds_ell = [&](int waves, bool ordered) {
    const size_t cap = ordered ? 2 * (size_t)w : 0;
    return (size_t)P.max_sub * 4 + waves * 2 * (P.max_sub + 2 * cap + (cap + 1) / 2);
  };
  bool ordered = true;
  int ell_waves = 4;
  while (lds_ell(ell_waves, ordered) > lds_max) {
    if (ell_waves > 1) {
      ell_waves /= 2;
    } else {
      ell_waves = 4;
      ordered = false;
    }
  }
  hipLaunchKernelGGL(k_foe_ell,
                     dim3(P.n_sub, ((P.max_sub + 1) / 2 + kPairsPerBlock - 1) / kPairsPerBlock),
                     dim3(64 * ell_waves), lds_ell(ell_waves, ordered), s,
                     H.col, H.val, w, emin, emax, P.core_ptr.get(),
                     P.sub_ptr.get(), P.sub_idx.get(), eoff.get(), npad.get(), idx, val,
                     len.get(), ordered ? 1 : 0);
  GB_LAUNCH_CHECK();
  GB_HIP(hipEventRecord(t_stage.b, s));
  GB_HIP(hipStreamSynchronize(s));
  st.ms_gather = elapsed(t_stage.a, t_stage.b);

  // a pair of columns per thread where a workgroup holds that many, else as few equal rounds as
  // possible
  const int waves = ((P.max_sub + 1) / 2 + 63) / 64, most = 16;
  const int rounds = (waves + most - 1) / most;
  const int threads = 64 * ((waves + rounds - 1) / rounds);
  const int ntr = (M + 1) / 2;  // products that give the traces t_1 .. t_M
  DBuf<double> part((size_t)n_items * 2 * ntr, s), sums(2 * (size_t)ntr, s), dc(M + 1, s), sp;
  if (spill) sp = DBuf<double>((size_t)n_items * P.max_sub, s);
  std::vector<double> traces(M + 1, 0.0), c(M + 1), h(2 * (size_t)ntr);
  Timer t_pass;
  auto pass = [&](const double* coef, int nterm, bool want_traces, double* hist, int t_from) {
    const size_t lds = spill ? (size_t)P.max_sub * 8 : lds_of(R);
    const int nt = want_traces ? ntr : 0;
    GB_HIP(hipEventRecord(t_pass.a, s));
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(n_items), dim3(threads), lds, s, ditems.get(), idx, val,
                         len.get(), eoff.get(), P.sub_ptr.get(), P.core_ptr.get(), soff.get(),
                         nterm, nt, coef, Dacc, part.get(), sp.get(), P.max_sub, hist, ts, t_from);
    };
    if (spill) launch(k_foe_rows<1, true>);
    else if (R == 4) launch(k_foe_rows<4, false>);
    else if (R == 2) launch(k_foe_rows<2, false>);
    else launch(k_foe_rows<1, false>);
    GB_LAUNCH_CHECK();
    GB_HIP(hipEventRecord(t_pass.b, s));
    if (want_traces) {
      hipLaunchKernelGGL(k_foe_sums, dim3(2 * ntr), dim3(kT), 0, s, part.get(), n_items, 2 * ntr,
                         sums.get());
      GB_LAUNCH_CHECK();
      GB_HIP(hipMemcpyAsync(h.data(), sums.get(), h.size() * 8, hipMemcpyDeviceToHost, s));
    }
    GB_HIP(hipStreamSynchronize(s));
    st.ms_product += elapsed(t_pass.a, t_pass.b);
    st.n_product += nterm - t_from - (t_from == 0);
    ++st.passes;
    if (!want_traces) return;
    traces[0] = t0;
    traces[1] = h[0];
    for (int n = 0; n < ntr; ++n) {
      if (n > 0) traces[2 * n + 1] = 2.0 * h[2 * n] - traces[1];
      if (2 * n + 2 <= M) traces[2 * n + 2] = 2.0 * h[2 * n + 1] - t0;
    }
  };

  GB_HIP(hipEventRecord(t_stage.a, s));
  const int K = quad_nodes(M, o.n_nodes);
  const double mid = 0.5 * (emax + emin), half = 0.5 * (emax - emin);
  double mu = o.mu;
  const bool solve = std::isnan(mu);
  std::unique_ptr<CachedBuf> hist;
  if (solve) {
    // the terms of the first pass are kept for the second where they fit
    const size_t need = (size_t)ntr * ts * 8;
    if (need <= kHistMost) {
      try {
        hist = std::make_unique<CachedBuf>(need, s);
      } catch (const Error&) {  // no memory for them: the second pass makes them again
      }
    }
    pass(nullptr, ntr, true, hist ? (double*)hist->p : nullptr, 0);
    DBuf<double> dt(M + 1, s), de(K, s), dw(K, s), dm(3, s);
    GB_HIP(hipMemcpyAsync(dt.get(), traces.data(), (M + 1) * 8, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_foe_nodes, dim3((K + kT / 64 - 1) / (kT / 64)), dim3(kT), 0, s, dt.get(),
                       M, K, mid, half, de.get(), dw.get());
    hipLaunchKernelGGL(k_foe_mu, dim3(1), dim3(960), 0, s, de.get(), dw.get(), K, emin, emax,
                       o.beta, (double)n_occ, dm.get());
    GB_LAUNCH_CHECK();
    double m[3];
    GB_HIP(hipMemcpyAsync(m, dm.get(), sizeof(m), hipMemcpyDeviceToHost, s));
    GB_HIP(hipStreamSynchronize(s));
    if (m[1] - n_occ > 0.0 || m[2] - n_occ < 0.0) fail_occupation(n_occ, m[1], m[2]);
    mu = m[0];
  }
  hipLaunchKernelGGL(k_foe_coef, dim3(M + 1), dim3(kT), 0, s, K, mid, half, o.beta, mu, dc.get());
  GB_LAUNCH_CHECK();
  GB_HIP(hipMemcpyAsync(c.data(), dc.get(), (M + 1) * 8, hipMemcpyDeviceToHost, s));
  pass(dc.get(), M, !solve, hist ? (double*)hist->p : nullptr, hist ? ntr : 0);
  GB_HIP(hipEventRecord(t_stage.b, s));
  GB_HIP(hipStreamSynchronize(s));
  st.ms_terms = elapsed(t_stage.a, t_stage.b);
  st.mu = mu;
  double tr = 0.0;
  for (int n = 0; n <= M; ++n) tr += c[n] * traces[n];
  st.trace = tr;
  st.coef_tail = std::fabs(c[M]) + std::fabs(c[M - 1]);
  if (o.traces) std::memcpy(o.traces, traces.data(), (M + 1) * sizeof(double));

  GB_HIP(hipEventRecord(t_stage.a, s));
  hipLaunchKernelGGL(k_scatter<double>, dim3(N), dim3(kT), 0, s, Dacc, soff.get(),
                     npad.get(), P.sub_ptr.get(), P.sub_idx.get(), P.sub_pos.get(),
                     P.col_sub.get(), P.col_loc.get(), D.width, D.col, D.val);
  GB_LAUNCH_CHECK();
  GB_HIP(hipEventRecord(t_stage.b, s));
  GB_HIP(hipEventRecord(t_all.b, s));
  GB_HIP(hipStreamSynchronize(s));
  st.ms_scatter = elapsed(t_stage.a, t_stage.b);
  st.ms_total += elapsed(t_all.a, t_all.b);
}

}  // namespace gbi
