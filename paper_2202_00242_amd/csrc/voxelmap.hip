// Voxel map of a target cloud (Sec. III-A): every voxel holds the arithmetic mean of its
// member points' means and covariances. Deterministic GPU build:
//   1. FP64 voxel coordinates of every point, range and finiteness checks, coordinate bounds;
//   2. a dense sort key (the coordinates relative to their minimum, packed with just enough
//      bits per axis so that key order is lexicographic (x, y, z) order);
//   3. a stable LSD radix sort of (key, point index) - members of a voxel stay in increasing
//      point index;
//   4. segment heads and an exclusive scan: voxel id = rank of the key (canonical, independent
//      of point order and of the hash layout);
//   5. per voxel, FP64 sums in increasing point index -> mean and covariance;
//   6. the voxel Gaussians in id order (80-byte records) and a lookup structure: occupancy
//      bricks of 4 x 4 x 2 voxels over the map's voxel bounding box (with a copy of the records
//      in brick order) when the box is moderate, else an open-addressing table of {key, id} slots (capacity a power of two >= 4 V,
//      linear probing), the key relative to the bounding box and 32-bit whenever the box needs
//      at most 31 bits.
#include <algorithm>
#include <cmath>
#include <vector>

#include "device_math.h"
#include "internal.h"
#include "sort.h"

namespace vgicp {
namespace {

constexpr int kBlock = 256;
constexpr int kItems = 8;
constexpr int kTile = kBlock * kItems;  // elements per block in scans and radix passes
constexpr long long kGridMaxBricks = 1LL << 24;   // 128 MiB of brick records (24-bit indexing)
constexpr long long kGridAutoBricks = 1LL << 23;  // 64 MiB of brick records

// ------------------------------------------------------------------ step 1: coordinates

__global__ __launch_bounds__(kBlock) void coords_kernel(const float* __restrict__ xyz,
                                                        const float* __restrict__ cov,
                                                        long long n, int pow2, double res,
                                                        double inv_res, int* __restrict__ kc,
                                                        int* __restrict__ bounds,
                                                        BuildReport* __restrict__ report) {
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
  unsigned fl = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    for (int a = 0; a < 6; ++a)
      if (!isfinite(cov[a * n + i])) fl |= kFlagNonFinite;
    for (int a = 0; a < 3; ++a) {
      int k = 0;
      const int st = pow2 ? voxel_coord<false>((double)xyz[a * n + i], res, inv_res, &k)
                          : voxel_coord<true>((double)xyz[a * n + i], res, inv_res, &k);
      if (st == 1) fl |= kFlagNonFinite;
      if (st == 2) fl |= kFlagKeyRange;
      kc[a * n + i] = k;
      lo[a] = min(lo[a], k);
      hi[a] = max(hi[a], k);
    }
  }
  for (int a = 0; a < 3; ++a) {
    for (int off = 32; off > 0; off >>= 1) {
      lo[a] = min(lo[a], __shfl_xor(lo[a], off, 64));
      hi[a] = max(hi[a], __shfl_xor(hi[a], off, 64));
    }
  }
  publish_bounds(lo, hi, bounds, report);
  if (fl & kFlagNonFinite) report->nonfinite = 1;
  if (fl & kFlagKeyRange) report->keyrange = 1;
}

// Start of a call: zeroed words (digit counts), the integer bounds with their ticket, the report.
__global__ __launch_bounds__(kBlock) void call_init_kernel(int* __restrict__ zero, long long words,
                                                           int* __restrict__ bounds,
                                                           BuildReport* __restrict__ report) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < words;
       i += (long long)gridDim.x * blockDim.x)
    zero[i] = 0;
  if (blockIdx.x == 0) {
    if (bounds && threadIdx.x < 7)
      bounds[threadIdx.x] = threadIdx.x < 3 ? INT_MAX : (threadIdx.x < 6 ? INT_MIN : 0);
    if (report)
      for (unsigned i = threadIdx.x; i < sizeof(BuildReport) / 4; i += blockDim.x)
        reinterpret_cast<int*>(report)[i] = 0;
  }
}

// ------------------------------------------------------------------ step 2: sort keys

// One block per sort tile; hist (may be null): the first pass's digit counts of every tile.
__global__ __launch_bounds__(kBlock) void sortkey_kernel(const int* __restrict__ kc, long long n,
                                                         int lx, int ly, int lz, int by, int bz,
                                                         unsigned long long* __restrict__ key,
                                                         int* __restrict__ val,
                                                         int* __restrict__ hist) {
  unsigned digit[kSortTile / kBlock];
  bool valid[kSortTile / kBlock];
#pragma unroll
  for (int j = 0; j < kSortTile / kBlock; ++j) {
    const long long i = (long long)blockIdx.x * kSortTile + j * kBlock + threadIdx.x;
    valid[j] = i < n;
    digit[j] = 0;
    if (!valid[j]) continue;
    const unsigned long long x = (unsigned long long)(kc[i] - lx);
    const unsigned long long y = (unsigned long long)(kc[n + i] - ly);
    const unsigned long long z = (unsigned long long)(kc[2 * n + i] - lz);
    const unsigned long long k = (x << (by + bz)) | (y << bz) | z;
    key[i] = k;
    val[i] = (int)i;
    digit[j] = (unsigned)k;
  }
  if (hist) sort_tile_hist(digit, valid, hist + (size_t)blockIdx.x * 256);
}

// ------------------------------------------------------------------ exclusive scan (int)

// Block-wide exclusive scan of kTile ints (thread t owns elements t*kItems..t*kItems+7 of the
// tile); in and out may be the same array. Writes each block's total to block_sums when it is
// not null.
__global__ __launch_bounds__(kBlock) void scan_tile_kernel(const int* in, int* out, long long n,
                                                           int* __restrict__ block_sums) {
  __shared__ int wsum[kBlock / 64];
  const long long base = (long long)blockIdx.x * kTile + (long long)threadIdx.x * kItems;
  int v[kItems];
  int run = 0;
  for (int k = 0; k < kItems; ++k) {
    const long long i = base + k;
    v[k] = (i < n) ? in[i] : 0;
    run += v[k];
  }
  // inclusive scan of thread totals within the wave
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = run;
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int before = 0;
  for (int k = 0; k < w; ++k) before += wsum[k];
  int excl = before + x - run;
  for (int k = 0; k < kItems; ++k) {
    const long long i = base + k;
    if (i < n) out[i] = excl;
    excl += v[k];
  }
  if (block_sums && threadIdx.x == kBlock - 1) block_sums[blockIdx.x] = before + x;
}

__global__ __launch_bounds__(kBlock) void scan_add_kernel(int* __restrict__ out, long long n,
                                                          const int* __restrict__ offs) {
  const long long base = (long long)blockIdx.x * kTile;
  const int o = offs[blockIdx.x];
  for (int k = threadIdx.x; k < kTile; k += kBlock) {
    const long long i = base + k;
    if (i < n) out[i] += o;
  }
}

// Exclusive scan of n ints (in -> out, may alias), recursive over block totals.
hipError_t exclusive_scan(const int* in, int* out, long long n, hipStream_t s, Scratch& sc) {
  if (n <= 0) return hipSuccess;
  const long long nb = (n + kTile - 1) / kTile;
  if (nb == 1) {
    scan_tile_kernel<<<1, kBlock, 0, s>>>(in, out, n, nullptr);
    return hipGetLastError();
  }
  int* sums = nullptr;
  hipError_t e = sc.alloc(&sums, (size_t)nb);
  if (e != hipSuccess) return e;
  scan_tile_kernel<<<(unsigned)nb, kBlock, 0, s>>>(in, out, n, sums);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = exclusive_scan(sums, sums, nb, s, sc)) != hipSuccess) return e;
  scan_add_kernel<<<(unsigned)nb, kBlock, 0, s>>>(out, n, sums);
  return hipGetLastError();
}

// ------------------------------------------------------------------ stable LSD radix sort

__global__ __launch_bounds__(kBlock) void radix_hist_kernel(
    const unsigned long long* __restrict__ key, long long n, int shift, int* __restrict__ hist,
    int ntiles) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const long long base = (long long)blockIdx.x * kTile;
  for (int r = 0; r < kItems; ++r) {
    const long long i = base + r * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[(int)((key[i] >> shift) & 255ull)], 1);
  }
  __syncthreads();
  hist[threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// Scatter of one 8-bit digit. The tile's items are visited in rounds r of kBlock consecutive
// elements; within a round, a lane's rank among equal digits comes from wave ballots and the
// per-wave counts of lower waves, so the output keeps input order among equal digits.
__global__ __launch_bounds__(kBlock) void radix_scatter_kernel(
    const unsigned long long* __restrict__ kin, const int* __restrict__ vin,
    unsigned long long* __restrict__ kout, int* __restrict__ vout, long long n, int shift,
    const int* __restrict__ offsets, int ntiles, int* __restrict__ internal) {
  __shared__ int running[256];
  __shared__ int wcount[kBlock / 64][256];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  running[t] = offsets[t * ntiles + blockIdx.x];
  const long long base = (long long)blockIdx.x * kTile;
  const unsigned long long lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
  for (int r = 0; r < kItems; ++r) {
    for (int j = t; j < (kBlock / 64) * 256; j += kBlock) (&wcount[0][0])[j] = 0;
    __syncthreads();
    const long long i = base + r * kBlock + t;
    const bool valid = i < n;
    const unsigned long long k = valid ? kin[i] : 0ull;
    const int v = valid ? vin[i] : 0;
    const int dgt = (int)((k >> shift) & 255ull);
    unsigned long long peers = __ballot(valid);
    for (int bit = 0; bit < 8; ++bit) {
      const bool set = (dgt >> bit) & 1;
      const unsigned long long m = __ballot(set);
      peers &= set ? m : ~m;
    }
    const int rank = __popcll(peers & lt);
    if (valid && rank == 0) wcount[w][dgt] = __popcll(peers);
    __syncthreads();
    if (valid) {
      int off = running[dgt] + rank;
      for (int ww = 0; ww < w; ++ww) off += wcount[ww][dgt];
      if (off >= 0 && off < n) {
        kout[off] = k;
        vout[off] = v;
      } else {
        *internal = 1;
      }
    }
    __syncthreads();
    int add = 0;
    for (int ww = 0; ww < kBlock / 64; ++ww) add += wcount[ww][t];
    running[t] += add;
    __syncthreads();
  }
}

// One pass of the sort up to kSortMax pairs: block (tile, segment). Its digits' destinations are the
// digit totals below, the predecessors' counts of the digit, and the rank within the tile (wave
// ballots over items in order). Adding up the predecessors is at most 256 coalesced rows of 1 KB, and
// spares the three launches of a scan (113,000 points: five launches and 25 us a pass before, two and
// 13 us now; counting the next pass's digits here, by atomics on the destination tile's row, took
// 16); beyond kSortMax the rows outgrow the keys.
__global__ __launch_bounds__(kBlock) void sort_pass_kernel(
    const unsigned long long* __restrict__ kin, const int* __restrict__ vin,
    unsigned long long* __restrict__ kout, int* __restrict__ vout,
    const SortSeg* __restrict__ segs, int n_one, int shift, int max_tiles,
    const int* __restrict__ hist, int* __restrict__ internal) {
  constexpr int J = kSortTile / kBlock;
  __shared__ int wcnt[kBlock / 64][256];
  const int seg = blockIdx.y, tile = blockIdx.x;
  const long long off = segs ? segs[seg].off : 0;
  const int n = segs ? segs[seg].n : n_one;
  if (tile * kSortTile >= n) return;
  const int ntiles = (n + kSortTile - 1) / kSortTile;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  for (int q = 0; q < kBlock / 64; ++q) wcnt[q][t] = 0;
  // thread t is digit t
  const int* h = hist + (size_t)seg * max_tiles * 256 + t;
  int before = 0, all = 0;
  int r = 0;
  for (; r < ntiles; r += 32) {  // 32 rows in flight: each comes from beyond this XCD's L2
    int c[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) c[q] = r + q < ntiles ? h[(size_t)(r + q) * 256] : 0;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      all += c[q];
      before += r + q < tile ? c[q] : 0;
    }
  }
  int total;
  const int digit_base = block_prefix_256(all, total) + before;
  // wave w ranks the items w * 256 .. + 255 of the tile, 64 at a time
  const unsigned long long lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
  unsigned long long key[J];
  int val[J], dgt[J], rank[J];
  bool valid[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = tile * kSortTile + w * (kSortTile / 4) + j * 64 + lane;
    valid[j] = i < n;
    key[j] = valid[j] ? kin[off + i] : 0ull;
    val[j] = valid[j] ? vin[off + i] : 0;
    dgt[j] = (int)((key[j] >> shift) & 255ull);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < J; ++j) {
    unsigned long long peers = __ballot(valid[j]);
    for (int bit = 0; bit < 8; ++bit) {
      const bool set = (dgt[j] >> bit) & 1;
      const unsigned long long m = __ballot(set);
      peers &= set ? m : ~m;
    }
    const int pos = __popcll(peers & lt);
    rank[j] = pos + (valid[j] ? wcnt[w][dgt[j]] : 0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (valid[j] && pos == 0) wcnt[w][dgt[j]] += __popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __syncthreads();
  int run = digit_base;
  for (int q = 0; q < kBlock / 64; ++q) {
    const int c = wcnt[q][t];
    wcnt[q][t] = run;
    run += c;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (!valid[j]) continue;
    const int dst = wcnt[w][dgt[j]] + rank[j];
    if (dst < 0 || dst >= n) {
      *internal = 1;
      continue;
    }
    kout[off + dst] = key[j];
    vout[off + dst] = val[j];
  }
}

// Digit counts of every tile for a pass after the first.
__global__ __launch_bounds__(kBlock) void sort_hist_kernel(
    const unsigned long long* __restrict__ key, const SortSeg* __restrict__ segs, int n_one,
    int shift, int max_tiles, int* __restrict__ hist) {
  const int n = segs ? segs[blockIdx.y].n : n_one;
  const long long off = segs ? segs[blockIdx.y].off : 0;
  if ((int)blockIdx.x * kSortTile >= n) return;
  unsigned digit[kSortTile / kBlock];
  bool valid[kSortTile / kBlock];
#pragma unroll
  for (int j = 0; j < kSortTile / kBlock; ++j) {
    const int i = blockIdx.x * kSortTile + j * kBlock + threadIdx.x;
    valid[j] = i < n;
    digit[j] = valid[j] ? (unsigned)(key[off + i] >> shift) : 0u;
  }
  sort_tile_hist(digit, valid, hist + ((size_t)blockIdx.y * max_tiles + blockIdx.x) * 256);
}

// ------------------------------------------------------------------ scans over at most kRunTiles blocks

// What a scan adds up: the heads of runs of equal keys, an int array, or the voxels of bricks.
struct RunHeads {
  const unsigned long long* key;
  int* start;
  long long n;
  __device__ int value(long long i) const { return i == 0 || key[i] != key[i - 1] ? 1 : 0; }
  __device__ void put(long long i, int base, int v) const {
    if (v) start[base] = (int)i;
  }
  __device__ void end(int total) const { start[total] = (int)n; }
};
struct Ints {
  const int* in;
  int* out;
  long long n;
  __device__ int value(long long i) const { return in[i]; }
  __device__ void put(long long i, int base, int) const { out[i] = base; }
  __device__ void end(int) const {}
};
struct BrickVoxels {
  Brick* b;
  long long n;
  __device__ int value(long long i) const { return __popc(b[i].mask); }
  __device__ void put(long long i, int base, int) const { b[i].base = base; }
  __device__ void end(int) const {}
};

// Two launches instead of three per level: a block's total, then every block adds up its
// predecessors' totals (at most kRunTiles, four loads a thread) and walks its items. Block b has the
// items b * per .. + per - 1 (per: a multiple of 1,024).
template <class Op>
__global__ __launch_bounds__(kBlock) void scan_total_kernel(Op op, long long per,
                                                            int* __restrict__ tile_counts) {
  const long long first = blockIdx.x * per, end = min(first + per, op.n);
  int v = 0;
  for (long long i = first + threadIdx.x; i < end; i += kBlock) v += op.value(i);
  const int total = block_total_256(v);
  if (threadIdx.x == 0) tile_counts[blockIdx.x] = total;
}

template <class Op>
__global__ __launch_bounds__(kBlock) void scan_put_kernel(Op op, long long per,
                                                          const int* __restrict__ tile_counts,
                                                          int* __restrict__ total_out) {
  int v = 0;
  for (int t = threadIdx.x; t < (int)blockIdx.x; t += kBlock) v += tile_counts[t];
  int run = block_total_256(v);
  const long long first = blockIdx.x * per, end = min(first + per, op.n);
  for (long long base = first; base < end; base += 1024) {
    const long long i0 = base + 4 * threadIdx.x;
    int x[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = i0 + j < end ? op.value(i0 + j) : 0;
      sum += x[j];
    }
    int total;
    int at = run + block_prefix_256(sum, total);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (i0 + j < end) op.put(i0 + j, at, x[j]);
      at += x[j];
    }
    run += total;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    op.end(run);
    if (total_out) *total_out = run;
  }
}

template <class Op>
hipError_t scan_with(Op op, int* tile_counts, int* total, hipStream_t s) {
  const long long units = std::max<long long>((op.n + 1023) / 1024, 1);
  const long long per = (units + kRunTiles - 1) / kRunTiles * 1024;
  const unsigned blocks = (unsigned)std::max<long long>((op.n + per - 1) / per, 1);
  scan_total_kernel<<<blocks, kBlock, 0, s>>>(op, per, tile_counts);
  scan_put_kernel<<<blocks, kBlock, 0, s>>>(op, per, tile_counts, total);
  return hipGetLastError();
}

// ------------------------------------------------------------------ steps 4-6

__device__ inline void voxel_box_coords(long long k, int lo0, int lo1, int lo2, unsigned& dx,
                                        unsigned& dy, unsigned& dz) {
  const int m21 = (1 << 21) - 1;
  dx = (unsigned)((int)((k >> 42) & m21) - (int)kKeyLimit - lo0);
  dy = (unsigned)((int)((k >> 21) & m21) - (int)kKeyLimit - lo1);
  dz = (unsigned)((int)(k & m21) - (int)kKeyLimit - lo2);
}

// FP64 sums over a voxel's members in increasing point index: 16 lanes per voxel, one of the 9
// components each (a thread per voxel held up its wave for the fullest of 64 voxels, 9 gathers a
// member: 22 us for 24,000 voxels), four members' loads in flight. With bricks the voxel sets its bit
// in its brick's occupancy mask (cleared before).
__global__ __launch_bounds__(kBlock) void stats_kernel(
    const float* __restrict__ xyz, const float* __restrict__ cov, long long n,
    const int* __restrict__ kc, const int* __restrict__ order,
    const unsigned long long* __restrict__ skey, const int* __restrict__ start, int V,
    long long* __restrict__ keys, unsigned* __restrict__ rkey, double* __restrict__ mean,
    double* __restrict__ vcov, int* __restrict__ count, VoxelData* __restrict__ vox,
    Brick* __restrict__ bricks, int lo0, int lo1, int lo2, int gby, int gbz,
    int* __restrict__ internal) {
  const int v = (int)(((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 4);
  const int c = threadIdx.x & 15;
  if (v >= V) return;
  const int s = start[v], e = start[v + 1];
  if (!(s >= 0 && s < e && e <= n)) {
    *internal = 1;
    return;
  }
  const double cnt = (double)(e - s);
  if (c < 9) {
    const float* plane = c < 3 ? xyz + (size_t)c * n : cov + (size_t)(c - 3) * n;
    double sum = 0.0;
    int k = s;
    bool bad = false;
    for (; k + 4 <= e; k += 4) {
      float x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = order[k + q];
        bad |= j < 0 || j >= n;
        x[q] = plane[bad ? 0 : j];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) sum += (double)x[q];
    }
    for (; k < e; ++k) {
      const int j = order[k];
      bad |= j < 0 || j >= n;
      sum += (double)plane[bad ? 0 : j];
    }
    if (bad) *internal = 1;
    const double r = sum / cnt;
    if (c < 3) {
      vox[v].mean[c] = r;
      mean[(long long)c * V + v] = r;
    } else {
      vox[v].cov[c - 3] = r;
      vcov[(long long)(c - 3) * V + v] = r;
    }
  } else if (c == 9) {
    const long long j0 = order[s];
    const int k0 = kc[j0], k1 = kc[n + j0], k2 = kc[2 * n + j0];
    const long long key = pack_key(k0, k1, k2);
    keys[v] = key;
    rkey[v] = (unsigned)skey[s];
    vox[v].count = e - s;
    vox[v].pad = 0;
    count[v] = e - s;
    if (bricks) {
      unsigned dx, dy, dz;
      voxel_box_coords(key, lo0, lo1, lo2, dx, dy, dz);
      atomicOr(&bricks[brick_of(dx, dy, dz, (unsigned)gby, (unsigned)gbz)].mask,
               1u << bit_in_brick(dx, dy, dz));
    }
  }
}

__global__ __launch_bounds__(kBlock) void slots32_init_kernel(uint2* __restrict__ t, long long cap) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < cap;
       i += (long long)gridDim.x * blockDim.x)
    t[i] = make_uint2(kEmpty32, 0xffffffffu);
}

__global__ __launch_bounds__(kBlock) void slots64_init_kernel(longlong2* __restrict__ t,
                                                              long long cap) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < cap;
       i += (long long)gridDim.x * blockDim.x) {
    longlong2 e;
    e.x = kEmpty64;
    e.y = -1;
    t[i] = e;
  }
}

// One thread per voxel; keys are distinct, so every insertion claims a fresh slot. The table
// keeps at least three quarters of its slots free, so the probe ends within capacity steps.
__global__ __launch_bounds__(kBlock) void insert32_kernel(const unsigned* __restrict__ rkey, int V,
                                                          uint2* __restrict__ t, unsigned mask) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  const unsigned k = rkey[v];
  unsigned slot = hash32(k) & mask;
  for (unsigned p = 0; p <= mask; ++p) {
    if (atomicCAS(&t[slot].x, kEmpty32, k) == kEmpty32) {
      t[slot].y = (unsigned)v;
      return;
    }
    slot = (slot + 1) & mask;
  }
}

__global__ __launch_bounds__(kBlock) void insert64_kernel(const long long* __restrict__ keys, int V,
                                                          longlong2* __restrict__ t,
                                                          unsigned mask) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  const long long k = keys[v];
  unsigned slot = hash64(k) & mask;
  for (unsigned p = 0; p <= mask; ++p) {
    unsigned long long* kp = reinterpret_cast<unsigned long long*>(&t[slot].x);
    if (atomicCAS(kp, (unsigned long long)kEmpty64, (unsigned long long)k) ==
        (unsigned long long)kEmpty64) {
      t[slot].y = v;
      return;
    }
    slot = (slot + 1) & mask;
  }
}

// Grid layout: one thread per voxel copies its record to its brick-ordered position.
__global__ __launch_bounds__(kBlock) void brick_place_kernel(
    const long long* __restrict__ keys, int V, int lo0, int lo1, int lo2, int gby, int gbz,
    const Brick* __restrict__ bricks, const VoxelData* __restrict__ vox,
    VoxelData* __restrict__ voxb, int* __restrict__ rec_id) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  unsigned dx, dy, dz;
  voxel_box_coords(keys[v], lo0, lo1, lo2, dx, dy, dz);
  const Brick br = bricks[brick_of(dx, dy, dz, (unsigned)gby, (unsigned)gbz)];
  const unsigned bit = bit_in_brick(dx, dy, dz);
  const int pos = br.base + __popc(br.mask & ((1u << bit) - 1u));
  voxb[pos] = vox[v];
  rec_id[pos] = v;
}

// ------------------------------------------------------------------ spatial order of a cloud

// What the kernels below read of a SpatialJob.
struct SpatialSeg {
  const float *xyz, *cov;
  float *xyz_out, *cov6_out;
  int* perm;
  long long off;
  double inv_cell;
  int n, box;  // box: index of the cloud's bounding box
};

// Bounding box of every cloud (grid: blocks x clouds): block minima and maxima, then the cloud's last
// block to arrive adds them up. A cloud with a coordinate that is not finite gets an infinite box
// (never skipped, so the kernels report it).
constexpr int kBoxBlocks = 16;
__global__ __launch_bounds__(kBlock) void cloud_boxes_kernel(const SpatialSeg* __restrict__ segs,
                                                             float* __restrict__ part,
                                                             int* __restrict__ tickets,
                                                             float* __restrict__ boxes) {
  __shared__ float red[7][kBlock / 64];
  __shared__ int s_last;
  const SpatialSeg g = segs[blockIdx.y];
  float v[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0f};
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < g.n; i += gridDim.x * kBlock)
    for (int a = 0; a < 3; ++a) {
      const float x = g.xyz[(size_t)a * g.n + i];
      if (!isfinite(x)) v[6] = 1.0f;
      v[a] = fminf(v[a], x);
      v[3 + a] = fmaxf(v[3 + a], x);
    }
  const int w = threadIdx.x >> 6;
  for (int a = 0; a < 7; ++a) {
    for (int off = 32; off > 0; off >>= 1) {
      const float o = __shfl_xor(v[a], off, 64);
      v[a] = a < 3 ? fminf(v[a], o) : fmaxf(v[a], o);
    }
    if ((threadIdx.x & 63) == 0) red[a][w] = v[a];
  }
  __syncthreads();
  float* mine = part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 8;
  if (threadIdx.x < 7) {
    float x = red[threadIdx.x][0];
    for (int q = 1; q < kBlock / 64; ++q)
      x = threadIdx.x < 3 ? fminf(x, red[threadIdx.x][q]) : fmaxf(x, red[threadIdx.x][q]);
    __hip_atomic_store(&mine[threadIdx.x], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(&tickets[blockIdx.y], 1) == (int)gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  if (threadIdx.x < 6) {
    const float* p = part + (size_t)blockIdx.y * gridDim.x * 8;
    float x = threadIdx.x < 3 ? INFINITY : -INFINITY, bad = 0.0f;
    for (unsigned q = 0; q < gridDim.x; ++q) {
      const float o = __hip_atomic_load(&p[q * 8 + threadIdx.x], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
      x = threadIdx.x < 3 ? fminf(x, o) : fmaxf(x, o);
      bad = fmaxf(bad, __hip_atomic_load(&p[q * 8 + 6], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT));
    }
    if (bad > 0.0f) x = threadIdx.x < 3 ? -INFINITY : INFINITY;
    boxes[6 * (size_t)g.box + threadIdx.x] = x;
  }
}

// Morton code of a point's cell: per axis u = floor(v / cell) + 2^20 clamped to 21 bits, bits
// interleaved x, y, z from the lowest. When every cell coordinate of the clouds lies in
// [-2^b, 2^b), bits 19 .. b of u repeat the complement of bit 20, so the code keeps bit 20 and
// the low b bits only: the order is the same (two codes that differ above bit b differ first at
// bit 20), in 3 (b + 1) bits instead of 63.
__global__ __launch_bounds__(kBlock) void morton_kernel(const SpatialSeg* __restrict__ segs, int b,
                                                        unsigned long long* __restrict__ code,
                                                        int* __restrict__ idx, int max_tiles,
                                                        int* __restrict__ hist) {
  const SpatialSeg g = segs[blockIdx.y];
  if ((long long)blockIdx.x * kSortTile >= g.n) return;
  unsigned digit[kSortTile / kBlock];
  bool valid[kSortTile / kBlock];
#pragma unroll
  for (int j = 0; j < kSortTile / kBlock; ++j) {
    const long long i = (long long)blockIdx.x * kSortTile + j * kBlock + threadIdx.x;
    valid[j] = i < g.n;
    digit[j] = 0;
    if (!valid[j]) continue;
    unsigned long long c = 0;
    for (int a = 0; a < 3; ++a) {
      double f = floor((double)g.xyz[(size_t)a * g.n + i] * g.inv_cell) + (double)kKeyLimit;
      f = fmin(fmax(f, 0.0), (double)(2 * kKeyLimit - 1));  // NaN -> 0
      const unsigned long long u = (unsigned long long)f;
      const unsigned long long low = b >= 20 ? u : ((u & ((1ull << b) - 1ull)) | ((u >> 20) << b));
      c |= spread3(low) << a;
    }
    code[g.off + i] = c;
    idx[g.off + i] = (int)i;
    digit[j] = (unsigned)c;
  }
  if (hist)
    sort_tile_hist(digit, valid, hist + ((size_t)blockIdx.y * max_tiles + blockIdx.x) * 256);
}

// Positions [3][n] and interleaved covariances [n][6] in the sorted order, and the order itself.
__global__ __launch_bounds__(kBlock) void gather_clouds_kernel(const SpatialSeg* __restrict__ segs,
                                                               const int* __restrict__ order,
                                                               int* __restrict__ internal) {
  const SpatialSeg g = segs[blockIdx.y];
  const size_t n = (size_t)g.n;
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < g.n;
       i += (long long)gridDim.x * kBlock) {
    const int j = order[g.off + i];
    if (j < 0 || j >= g.n) {
      *internal = 1;
      continue;
    }
    for (int a = 0; a < 3; ++a) g.xyz_out[a * n + i] = g.xyz[a * n + j];
    float2* o = reinterpret_cast<float2*>(g.cov6_out) + 3 * i;
    o[0] = make_float2(g.cov[j], g.cov[n + j]);
    o[1] = make_float2(g.cov[2 * n + j], g.cov[3 * n + j]);
    o[2] = make_float2(g.cov[4 * n + j], g.cov[5 * n + j]);
    g.perm[i] = j;
  }
}

int grid_for(long long n) {
  return (int)std::max<long long>(1, std::min<long long>((n + kBlock - 1) / kBlock, 65536));
}

int bits_for(long long span) {  // bits to hold values 0..span
  int b = 0;
  while ((1LL << b) <= span) ++b;
  return b;
}

}  // namespace

hipError_t radix_sort_pairs(unsigned long long** k, int** v, unsigned long long** kt, int** vt,
                            long long n, int bits, int* internal, hipStream_t s, Scratch& sc) {
  if (n <= 0) return hipSuccess;
  const long long ntiles = (n + kTile - 1) / kTile;
  int* hist = nullptr;
  hipError_t e = sc.alloc(&hist, (size_t)(256 * ntiles));
  if (e != hipSuccess) return e;
  for (int shift = 0; shift < bits; shift += 8) {
    radix_hist_kernel<<<(unsigned)ntiles, kBlock, 0, s>>>(*k, n, shift, hist, (int)ntiles);
    if ((e = exclusive_scan(hist, hist, 256 * ntiles, s, sc)) != hipSuccess) return e;
    radix_scatter_kernel<<<(unsigned)ntiles, kBlock, 0, s>>>(*k, *v, *kt, *vt, n, shift, hist,
                                                             (int)ntiles, internal);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    std::swap(*k, *kt);
    std::swap(*v, *vt);
  }
  return hipSuccess;
}

hipError_t sort_passes(SortBuffers& b, const SortSeg* segs, int nseg, long long max_n, int bits,
                       int* internal, hipStream_t s) {
  const int tiles = (int)sort_tiles(max_n), passes = (bits + 7) / 8;
  const dim3 grid((unsigned)tiles, (unsigned)nseg);
  for (int p = 0; p < passes; ++p) {
    if (p > 0)
      sort_hist_kernel<<<grid, kBlock, 0, s>>>(b.k, segs, (int)max_n, 8 * p, tiles, b.hist);
    sort_pass_kernel<<<grid, kBlock, 0, s>>>(b.k, b.v, b.kt, b.vt, segs, (int)max_n, 8 * p, tiles,
                                             b.hist, internal);
    std::swap(b.k, b.kt);
    std::swap(b.v, b.vt);
  }
  return hipGetLastError();
}

hipError_t run_starts(const unsigned long long* key, long long n, int* start, int* tile_counts,
                      int* count_out, hipStream_t s) {
  return scan_with(RunHeads{key, start, n}, tile_counts, count_out, s);
}

hipError_t scan_values(const int* in, int* out, long long n, int* tile_counts, int* total,
                       hipStream_t s) {
  return scan_with(Ints{in, out, n}, tile_counts, total, s);
}

void launch_call_init(int* zero, long long words, int* bounds, BuildReport* report,
                      hipStream_t s) {
  const unsigned blocks = (unsigned)std::max<long long>(1, std::min<long long>((words + 1023) / 1024, 1024));
  call_init_kernel<<<blocks, kBlock, 0, s>>>(zero, words, bounds, report);
}

vgicp_status spatial_copies(std::vector<SpatialJob>& jobs, float* d_boxes, hipStream_t s) {
  hipError_t e;
  const size_t C = jobs.size();
  if (C == 0) return VGICP_OK;
  // the clouds that factors read, the largest first: a group's digit counts and grid are those of its
  // largest cloud for every cloud in it
  std::vector<SpatialSeg> segs;
  for (size_t c = 0; c < C; ++c) {
    const SpatialJob& j = jobs[c];
    if (j.cell > 0.0)
      segs.push_back({j.xyz, j.cov, j.xyz_out, j.cov6_out, j.perm, 0, 1.0 / j.cell, (int)j.n,
                      (int)c});
  }
  std::stable_sort(segs.begin(), segs.end(),
                   [](const SpatialSeg& a, const SpatialSeg& b) { return a.n > b.n; });
  HostBlock hb;
  if (!hb.p) return fail(VGICP_E_OOM, "pinned host block");
  BuildReport* rep = static_cast<BuildReport*>(hb.p);
  const int S = (int)segs.size();
  std::vector<float> boxes(6 * C, 0.0f);
  Arena a0(&hb);
  a0.need<SpatialSeg>((size_t)S);
  a0.need<float>((size_t)S * kBoxBlocks * 8);
  a0.need<int>((size_t)S);
  if ((e = a0.get(s))) return hip_fail(e, "device block (cloud order)");
  SpatialSeg* d_segs = a0.take<SpatialSeg>((size_t)S);
  float* part = a0.take<float>((size_t)S * kBoxBlocks * 8);
  int* tickets = a0.take<int>((size_t)S);
  launch_call_init(reinterpret_cast<int*>(d_boxes), 6 * (long long)C, nullptr, rep, s);
  if (S > 0) {
    if ((e = hipMemcpyAsync(d_segs, segs.data(), (size_t)S * sizeof(SpatialSeg),
                            hipMemcpyHostToDevice, s)))
      return hip_fail(e, "cloud order");
    launch_call_init(tickets, S, nullptr, nullptr, s);
    for (int first = 0; first < S; first += 32768) {
      const int m = std::min(S - first, 32768);
      cloud_boxes_kernel<<<dim3(kBoxBlocks, (unsigned)m), kBlock, 0, s>>>(
          d_segs + first, part + (size_t)first * kBoxBlocks * 8, tickets + first, d_boxes);
    }
    if ((e = hipGetLastError()) ||
        (e = hipMemcpyAsync(boxes.data(), d_boxes, boxes.size() * sizeof(float),
                            hipMemcpyDeviceToHost, s)) ||
        (e = hipStreamSynchronize(s)))
      return hip_fail(e, "cloud boxes");
  }
  // bits of a cloud's cell coordinates: all in [-2^b, 2^b)
  auto bits_of = [&](const SpatialSeg& g) {
    int b = 0;
    for (int a = 0; a < 3; ++a) {
      const double lo = std::floor((double)boxes[6 * (size_t)g.box + a] * g.inv_cell);
      const double hi = std::floor((double)boxes[6 * (size_t)g.box + 3 + a] * g.inv_cell);
      while (b < 20 && !(lo >= -std::ldexp(1.0, b) && hi < std::ldexp(1.0, b))) ++b;
    }
    return b;
  };
  for (int first = 0; first < S;) {
    // as many clouds together as fit 4 M points (24 bytes each for their pairs: 96 MiB) and 2^16 tiles
    // of the largest (1 KB of digit counts each: 64 MiB). Clouds of one size reach the second bound
    // only where a cloud is far smaller than a tile (32,768 single points: 32 MiB); without it a cloud of
    // 2^18 points among 4,000 of 900 made 1 GB of counts.
    constexpr long long kGroupPoints = 4LL << 20, kGroupTiles = 1LL << 16;
    long long pts = 0, max_n = 1;
    int m = 0, b = 0;
    bool big = false;
    while (first + m < S && m < 32768) {
      SpatialSeg& g = segs[first + m];
      if (m > 0 && (big || g.n > kSortMax || pts + g.n > kGroupPoints ||
                    (m + 1) * sort_tiles(std::max<long long>(max_n, g.n)) > kGroupTiles))
        break;
      big = g.n > kSortMax;
      g.off = pts;
      pts += g.n;
      if (g.n > 0) b = std::max(b, bits_of(g));
      max_n = std::max<long long>(max_n, g.n);
      ++m;
    }
    const int bits = b >= 20 ? 63 : 3 * (b + 1);
    const long long tiles = sort_tiles(max_n);
    const size_t words = big ? 0 : sort_hist_ints(m, max_n);
    std::vector<SortSeg> ss;  // read by a copy until the stream is waited for, at the latest by the block
    for (int i = 0; i < m; ++i) ss.push_back({segs[first + i].off, segs[first + i].n, 0});
    Arena ar(&hb);
    Scratch sc;
    ar.need<unsigned long long>((size_t)pts);
    ar.need<unsigned long long>((size_t)pts);
    ar.need<int>((size_t)pts);
    ar.need<int>((size_t)pts);
    ar.need<int>(words);
    ar.need<SortSeg>((size_t)m);
    if ((e = ar.get(s))) return hip_fail(e, "device block (cloud order)");
    SortBuffers sb;
    sb.k = ar.take<unsigned long long>((size_t)pts);
    sb.kt = ar.take<unsigned long long>((size_t)pts);
    sb.v = ar.take<int>((size_t)pts);
    sb.vt = ar.take<int>((size_t)pts);
    sb.hist = ar.take<int>(words);
    SortSeg* d_ss = ar.take<SortSeg>((size_t)m);
    if ((e = hipMemcpyAsync(d_segs + first, segs.data() + first, (size_t)m * sizeof(SpatialSeg),
                            hipMemcpyHostToDevice, s)) ||
        (e = hipMemcpyAsync(d_ss, ss.data(), ss.size() * sizeof(SortSeg), hipMemcpyHostToDevice,
                            s)))
      return hip_fail(e, "cloud order");
    morton_kernel<<<dim3((unsigned)tiles, (unsigned)m), kBlock, 0, s>>>(
        d_segs + first, b, sb.k, sb.v, (int)tiles, big ? nullptr : sb.hist);
    if (big)
      e = radix_sort_pairs(&sb.k, &sb.v, &sb.kt, &sb.vt, pts, bits, &rep->internal, s, sc);
    else
      e = sort_passes(sb, d_ss, m, max_n, bits, &rep->internal, s);
    if (e) return hip_fail(e, "radix sort (cloud order)");
    gather_clouds_kernel<<<dim3((unsigned)std::min<long long>((max_n + 255) / 256, 4096),
                                (unsigned)m),
                           kBlock, 0, s>>>(d_segs + first, sb.v, &rep->internal);
    if ((e = hipGetLastError()) || (e = hipStreamSynchronize(s)))
      return hip_fail(e, "cloud order");
    first += m;
  }
  if ((e = hipStreamSynchronize(s))) return hip_fail(e, "cloud order");
  if (rep->internal) return fail(VGICP_E_HIP, "internal error in the cloud order");
  return VGICP_OK;
}

vgicp_status build_voxelmap(const float* xyz, const float* cov, int64_t n, double res,
                            int layout, hipStream_t s, vgicp_voxelmap* out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  auto* m = new vgicp_voxelmap_s;
  m->device = dev;
  m->res = res;
  m->inv_res = 1.0 / res;
  int ex = 0;
  m->pow2 = (std::frexp(res, &ex) == 0.5) ? 1 : 0;
  auto cleanup = [&](vgicp_status st) {
    destroy_voxelmap(m);
    return st;
  };
  HostBlock hb;
  if (!hb.p) return cleanup(fail(VGICP_E_OOM, "pinned host block"));
  volatile BuildReport* rep = static_cast<BuildReport*>(hb.p);
  BuildReport* report = static_cast<BuildReport*>(hb.p);
  // a pass of the sort is two launches up to kSortMax points (63 key bits: 8 passes)
  const bool small = n <= kSortMax;
  const size_t n1 = (size_t)std::max<int64_t>(n, 1);
  const size_t words = small && n > 0 ? sort_hist_ints(1, n) : 0;
  Arena ar(&hb);
  Scratch sc;
  ar.need<int>(3 * n1);
  ar.need<int>(8);
  ar.need<int>(words);
  ar.need<unsigned long long>(n1);
  ar.need<unsigned long long>(n1);
  ar.need<int>(n1);
  ar.need<int>(n1);
  ar.need<int>(n1 + 1);
  ar.need<unsigned>(n1);
  ar.need<int>(kRunTiles);
  if ((e = ar.get(s)) != hipSuccess) return cleanup(hip_fail(e, "voxel map scratch"));
  int* kc = ar.take<int>(3 * n1);
  int* bounds = ar.take<int>(8);
  SortBuffers sb;
  sb.hist = ar.take<int>(words);
  sb.k = ar.take<unsigned long long>(n1);
  sb.kt = ar.take<unsigned long long>(n1);
  sb.v = ar.take<int>(n1);
  sb.vt = ar.take<int>(n1);
  int* start = ar.take<int>(n1 + 1);
  unsigned* rkey = ar.take<unsigned>(n1);
  int* tile_counts = ar.take<int>(kRunTiles);
  launch_call_init(nullptr, 0, bounds, report, s);
  if (n > 0)
    coords_kernel<<<std::min(grid_for(n), 128), kBlock, 0, s>>>(xyz, cov, n, m->pow2, res,
                                                                m->inv_res, kc, bounds, report);
  if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess)
    return cleanup(hip_fail(e, "voxel coordinates"));
  if (rep->nonfinite) return cleanup(fail(VGICP_E_NONFINITE, "non-finite map point"));
  if (rep->keyrange)
    return cleanup(fail(VGICP_E_KEY_RANGE, "map point outside the voxel key range |k| < 2^20"));

  long long V = 0;
  int bits = 0;
  if (n > 0) {
    const int b[3] = {bits_for((long long)rep->hi[0] - rep->lo[0]),
                      bits_for((long long)rep->hi[1] - rep->lo[1]),
                      bits_for((long long)rep->hi[2] - rep->lo[2])};
    bits = b[0] + b[1] + b[2];  // <= 63
    for (int a = 0; a < 3; ++a) {
      m->lo[a] = rep->lo[a];
      m->ext[a] = rep->hi[a] - rep->lo[a] + 1;
    }
    m->by = b[1];
    m->bz = b[2];
    m->key32 = bits <= 31;
    if ((n + kTile - 1) / kTile * 256 >= (1LL << 31))
      return cleanup(fail(VGICP_E_CAPACITY, "map too large for the 32-bit sort offsets"));
    sortkey_kernel<<<(unsigned)sort_tiles(n), kBlock, 0, s>>>(
        kc, n, m->lo[0], m->lo[1], m->lo[2], b[1], b[2], sb.k, sb.v, small ? sb.hist : nullptr);
    e = small ? sort_passes(sb, nullptr, 1, n, bits, &report->internal, s)
              : radix_sort_pairs(&sb.k, &sb.v, &sb.kt, &sb.vt, n, bits, &report->internal, s, sc);
    if (e != hipSuccess) return cleanup(hip_fail(e, "radix sort"));
    if ((e = run_starts(sb.k, n, start, tile_counts, &report->count, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
      return cleanup(hip_fail(e, "voxel count"));
    V = rep->count;
    if (V <= 0 || V > n || rep->internal)
      return cleanup(fail(VGICP_E_HIP, "internal error: voxel count"));
    m->V = V;
  }
  // Grid layout: occupancy bricks of 4 x 4 x 2 voxels over the bounding box. The automatic
  // choice takes it while it needs at most kGridAutoBricks bricks or 32 per voxel; else the
  // hash table.
  const long long gbx = ((long long)m->ext[0] + 3) / 4, gby = ((long long)m->ext[1] + 3) / 4,
                  gbz = ((long long)m->ext[2] + 1) / 2;
  const long long nb = (n > 0) ? gbx * gby * gbz : 0;
  bool use_grid = false;
  if (layout == VGICP_LAYOUT_GRID) {
    if (nb > kGridMaxBricks)
      return cleanup(fail(VGICP_E_CAPACITY, "voxel grid above 2^24 bricks; use the hash layout"));
    use_grid = true;
  } else if (layout == VGICP_LAYOUT_AUTO) {
    use_grid = nb <= kGridMaxBricks && (nb <= kGridAutoBricks || nb <= 32 * V);
  }
  long long cap = 16;
  while (cap < 4 * V) cap <<= 1;
  if (cap > (1LL << 31)) return cleanup(fail(VGICP_E_CAPACITY, "voxel table above 2^31 slots"));
  m->layout = use_grid ? kLayoutGrid : (m->key32 ? kLayoutHash32 : kLayoutHash64);
  m->cap = use_grid ? 0 : cap;
  if (use_grid) {
    m->gby = (int)gby;
    m->gbz = (int)gbz;
    m->nbricks = std::max<long long>(nb, 1);
  }
  // the map's arrays, one block
  const size_t V1 = (size_t)std::max<long long>(V, 1);
  const size_t slot_bytes = use_grid ? 0 : (size_t)cap * (m->key32 ? sizeof(uint2) : sizeof(longlong2));
  Arena own;
  own.need<int64_t>(V1);
  own.need<double>(3 * V1);
  own.need<double>(6 * V1);
  own.need<int32_t>(V1);
  own.need<VoxelData>(V1);
  own.need<Brick>(use_grid ? (size_t)m->nbricks : 0);
  own.need<VoxelData>(use_grid ? V1 : 0);
  own.need<int>(use_grid ? V1 : 0);
  own.need<char>(slot_bytes);
  if ((e = own.get(s)) != hipSuccess) return cleanup(fail(VGICP_E_OOM, "voxel map arrays"));
  m->keys = own.take<int64_t>(V1);
  m->mean = own.take<double>(3 * V1);
  m->cov = own.take<double>(6 * V1);
  m->count = own.take<int32_t>(V1);
  m->vox = own.take<VoxelData>(V1);
  Brick* bricks = own.take<Brick>(use_grid ? (size_t)m->nbricks : 0);
  VoxelData* voxb = own.take<VoxelData>(use_grid ? V1 : 0);
  int* rec_id = own.take<int>(use_grid ? V1 : 0);
  char* slots = own.take<char>(slot_bytes);
  m->arena = own.keep(&m->arena_bytes);
  const long long* keys = reinterpret_cast<const long long*>(m->keys);
  const unsigned vb = (unsigned)((V1 + kBlock - 1) / kBlock);
  if (use_grid) {
    m->bricks = bricks;
    m->voxb = voxb;
    m->rec_id = rec_id;
    launch_call_init(reinterpret_cast<int*>(bricks), 2 * m->nbricks, nullptr, nullptr, s);
  } else if (m->key32) {
    m->slots32 = reinterpret_cast<uint2*>(slots);
    slots32_init_kernel<<<grid_for(cap), kBlock, 0, s>>>(m->slots32, cap);
  } else {
    m->slots64 = reinterpret_cast<longlong2*>(slots);
    slots64_init_kernel<<<grid_for(cap), kBlock, 0, s>>>(m->slots64, cap);
  }
  if (V > 0) {
    stats_kernel<<<(unsigned)((V + 15) / 16), kBlock, 0, s>>>(
        xyz, cov, n, kc, sb.v, sb.k, start, (int)V, reinterpret_cast<long long*>(m->keys), rkey,
        m->mean, m->cov, m->count, m->vox, m->bricks, m->lo[0], m->lo[1], m->lo[2], (int)gby,
        (int)gbz, &report->internal);
    if (use_grid) {
      if ((e = scan_with(BrickVoxels{m->bricks, nb}, tile_counts, nullptr, s)) != hipSuccess)
        return cleanup(hip_fail(e, "brick scan"));
      brick_place_kernel<<<vb, kBlock, 0, s>>>(keys, (int)V, m->lo[0], m->lo[1], m->lo[2],
                                               (int)gby, (int)gbz, m->bricks, m->vox, m->voxb,
                                               m->rec_id);
    } else if (m->key32) {
      insert32_kernel<<<vb, kBlock, 0, s>>>(rkey, (int)V, m->slots32, (unsigned)(cap - 1));
    } else {
      insert64_kernel<<<vb, kBlock, 0, s>>>(keys, (int)V, m->slots64, (unsigned)(cap - 1));
    }
  }
  if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess)
    return cleanup(hip_fail(e, "voxel table"));
  if (rep->internal) return cleanup(fail(VGICP_E_HIP, "internal error in the voxel map build"));
  *out = m;
  return VGICP_OK;
}

void destroy_voxelmap(vgicp_voxelmap m) {
  if (!m) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != m->device) (void)hipSetDevice(m->device);
  const hipError_t waited = hipDeviceSynchronize();
  if (m->arena) block_settle(m->arena, m->arena_bytes, m->device, waited);
  if (cur != m->device) (void)hipSetDevice(cur);
  delete m;
}

}  // namespace vgicp
