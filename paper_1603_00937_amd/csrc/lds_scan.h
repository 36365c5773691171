// Block-wide exclusive prefix sum of an int32 array held in LDS, shared by the graph and partition
// kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gbi {

// Inclusive prefix sum of x over the block's NT threads (whole waves), and the total.  Each wave
// scans by lane shifts, the waves' sums go through red (NT / 64 entries, free once every thread has
// passed the caller's next barrier): two barriers, where a scan of NT entries in LDS takes 2 log2
// NT.
template <int NT>
__device__ __forceinline__ int32_t block_inclusive_scan(int32_t x, int32_t* red, int32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  __syncthreads();
  if (lane == 63) red[wave] = x;
  __syncthreads();
  int32_t base = 0, tot = 0;
#pragma unroll
  for (int q = 0; q < NT / 64; ++q) {
    const int32_t r = red[q];
    if (q < wave) base += r;
    tot += r;
  }
  *total = tot;
  return base + x;
}

// v[0..m) <- exclusive prefix sums of v (in place); returns the total.  All NT threads of the
// block call it; red is an LDS array of at least NT / 64 entries.  Thread t owns the contiguous
// segment [t s, t s + s) of v, s = ceil(m / NT): segment sums, one scan of the NT sums, then each
// segment rewritten from its offset (one scan however long v is).
template <int NT>
__device__ __forceinline__ int32_t lds_exclusive_scan(int32_t* v, int m, int32_t* red) {
  const int seg = (m + NT - 1) / NT;
  const int b = min((int)threadIdx.x * seg, m), e = min(b + seg, m);
  int32_t sum = 0;
  for (int k = b; k < e; ++k) sum += v[k];
  int32_t total;
  int32_t run = block_inclusive_scan<NT>(sum, red, &total) - sum;
  for (int k = b; k < e; ++k) {
    const int32_t x = v[k];
    v[k] = run;
    run += x;
  }
  __syncthreads();
  return total;
}

}  // namespace gbi
