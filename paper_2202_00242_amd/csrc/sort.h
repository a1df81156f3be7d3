// Device side of the radix sort of two launches a pass (see SortBuffers in internal.h), and block sums.
#pragma once

#include "internal.h"

namespace vgicp {

// Digit counts of one tile for the first pass, by the block of 256 threads that made its keys:
// thread t's item j is item j * 256 + t of the tile. Every thread must call it.
__device__ inline void sort_tile_hist(const unsigned (&digit)[kSortTile / 256],
                                      const bool (&valid)[kSortTile / 256], int* __restrict__ out) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSortTile / 256; ++j)
    if (valid[j]) atomicAdd(&h[digit[j] & 255u], 1);
  __syncthreads();
  out[threadIdx.x] = h[threadIdx.x];
}

// Sum over the block's 256 threads of one int each, to all of them.
__device__ inline int block_total_256(int v) {
  __shared__ int sh[4];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Exclusive prefix of the block's 256 threads (one int each) and the total.
__device__ inline int block_prefix_256(int v, int& total) {
  __shared__ int sh[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  __syncthreads();
  if (lane == 63) sh[w] = x;
  __syncthreads();
  int before = 0;
  for (int k = 0; k < 4; ++k) before += k < w ? sh[k] : 0;
  total = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  return before + x - v;
}

// Integer bounds over a grid: one set of atomics per block (same-address atomics from every wave
// serialize), then the last block to arrive writes them to the report. bounds: 3 minima, 3 maxima,
// the ticket. Every thread must call it.
__device__ inline void publish_bounds(int (&lo)[3], int (&hi)[3], int* __restrict__ bounds,
                                      BuildReport* __restrict__ report) {
  __shared__ int red[6][16];
  const int w = threadIdx.x >> 6;
  for (int a = 0; a < 3; ++a)
    for (int off = 32; off > 0; off >>= 1) {
      lo[a] = min(lo[a], __shfl_xor(lo[a], off, 64));
      hi[a] = max(hi[a], __shfl_xor(hi[a], off, 64));
    }
  if ((threadIdx.x & 63) == 0)
    for (int a = 0; a < 3; ++a) {
      red[a][w] = lo[a];
      red[3 + a][w] = hi[a];
    }
  __syncthreads();
  if (threadIdx.x < 6) {
    int v = red[threadIdx.x][0];
    for (unsigned q = 1; q < blockDim.x / 64; ++q)
      v = threadIdx.x < 3 ? min(v, red[threadIdx.x][q]) : max(v, red[threadIdx.x][q]);
    if (threadIdx.x < 3)
      atomicMin(&bounds[threadIdx.x], v);
    else
      atomicMax(&bounds[threadIdx.x], v);
    __threadfence();
  }
  __syncthreads();
  __shared__ int last;
  if (threadIdx.x == 0) last = atomicAdd(&bounds[6], 1) == (int)gridDim.x - 1;
  __syncthreads();
  if (last && threadIdx.x < 6) {
    __threadfence();
    const int v = __hip_atomic_load(&bounds[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    (threadIdx.x < 3 ? report->lo[threadIdx.x] : report->hi[threadIdx.x - 3]) = v;
  }
}

}  // namespace vgicp
