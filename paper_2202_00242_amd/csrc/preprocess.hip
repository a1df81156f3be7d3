// Preprocessing of Sec. III-C on the GPU:
//   * voxel-grid filter: one output point per voxel, the FP64 mean of its members' positions
//     (and timestamps); with timestamps, a cell's points are taken in time order and a point
//     whose timestamp leaves the running mean timestamp of the cell's current voxel by more than
//     a tenth of the scan duration starts a new voxel of that cell, so that the first and last
//     points of a sweep do not fuse;
//   * the k nearest neighbours of every point (exact, ties by the lower index): uniform grid of
//     power-of-two cells over the Morton-sorted cloud, a hash of the occupied cells, and per
//     point a search over growing cubic shells of cells that stops once the k-th distance is
//     below the distance to the unsearched space;
//   * the point covariances C_k of Sec. III-A from those neighbours, plane-regularized as in
//     GICP (the eigenvalues of the neighbours' scatter replaced by scale * (1, 1, eps)).
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <vector>

#include "device_math.h"
#include "internal.h"
#include "sort.h"

namespace vgicp {
namespace {

constexpr int kBlock = 256;
constexpr unsigned long long kEmptyCell = ~0ull;

int grid_for(long long n) {
  return (int)std::max<long long>(1, std::min<long long>((n + kBlock - 1) / kBlock, 65536));
}

int bits_for(long long span) {  // bits to hold values 0..span
  int b = 0;
  while ((1LL << b) <= span) ++b;
  return b;
}

// ------------------------------------------------------------------ voxel-grid filter

// Cells floor(p / res) per axis in FP64 (a multiply for a power-of-two res, where it is exact),
// their bounds, and the finiteness / range checks of positions and timestamps.
__global__ __launch_bounds__(kBlock) void ds_cells_kernel(const float* __restrict__ xyz,
                                                          const float* __restrict__ t,
                                                          long long n, int pow2, double res,
                                                          double inv_res, int* __restrict__ kc,
                                                          int* __restrict__ bounds,
                                                          BuildReport* __restrict__ report) {
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
  unsigned fl = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    if (t && !isfinite(t[i])) fl |= kFlagNonFinite;
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
  publish_bounds(lo, hi, bounds, report);
  if (fl & kFlagNonFinite) report->nonfinite = 1;
  if (fl & kFlagKeyRange) report->keyrange = 1;
}

// Sort key of a timestamp: its FP32 bits made monotone as unsigned (-0 counted as +0). One block per
// sort tile; hist (may be null): the first pass's digit counts.
__global__ __launch_bounds__(kBlock) void ds_time_key_kernel(const float* __restrict__ t,
                                                             long long n,
                                                             unsigned long long* __restrict__ key,
                                                             int* __restrict__ idx,
                                                             int* __restrict__ hist) {
  unsigned digit[kSortTile / kBlock];
  bool valid[kSortTile / kBlock];
#pragma unroll
  for (int q = 0; q < kSortTile / kBlock; ++q) {
    const long long i = (long long)blockIdx.x * kSortTile + q * kBlock + threadIdx.x;
    valid[q] = i < n;
    digit[q] = 0;
    if (!valid[q]) continue;
    unsigned b = __float_as_uint(t[i] + 0.0f);
    b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    key[i] = b;
    idx[i] = (int)i;
    digit[q] = b;
  }
  if (hist) sort_tile_hist(digit, valid, hist + (size_t)blockIdx.x * 256);
}

// Cell key of the point at each position of `order` (identity if null): coordinates relative to
// the bounds, packed x-major so that key order is (x, y, z) lexicographic order. One block per sort
// tile; hist (may be null): the first pass's digit counts.
__global__ __launch_bounds__(kBlock) void ds_cell_key_kernel(const int* __restrict__ kc,
                                                             long long n,
                                                             const int* __restrict__ order,
                                                             int lx, int ly, int lz, int sy,
                                                             int sz,
                                                             unsigned long long* __restrict__ key,
                                                             int* __restrict__ val,
                                                             int* __restrict__ hist) {
  unsigned digit[kSortTile / kBlock];
  bool valid[kSortTile / kBlock];
#pragma unroll
  for (int q = 0; q < kSortTile / kBlock; ++q) {
    const long long i = (long long)blockIdx.x * kSortTile + q * kBlock + threadIdx.x;
    valid[q] = i < n;
    digit[q] = 0;
    if (!valid[q]) continue;
    const long long j = order ? order[i] : i;
    const unsigned long long k = ((unsigned long long)(kc[j] - lx) << sy) |
                                 ((unsigned long long)(kc[n + j] - ly) << sz) |
                                 (unsigned long long)(kc[2 * n + j] - lz);
    key[i] = k;
    val[i] = (int)j;
    digit[q] = (unsigned)k;
  }
  if (hist) sort_tile_hist(digit, valid, hist + (size_t)blockIdx.x * 256);
}

// Time order within the cells: a point's place is the number of its cell's points before it in
// (timestamp, index) order, counted directly (a cell holds a few points: for a sweep of 53,000
// points one launch of a few us instead of four passes of a sort by time). The block's 256 positions
// span few cells, whose timestamps go through LDS kRankChunk at a time. A cell costs its square: with
// 260,000 points in cells of 1,024 the ranks take 108 us and in cells of 4,000 347, the sort by time 88
// and 66 more for sorting by cell again, so a cell of more than kMaxRanked points sends the call there
// (cells of 2,000 to 8,192 points: 2.3, 4.1 and 8.0 ms for the filter, most of it the walks).
constexpr int kMaxRanked = 2048, kRankChunk = 1024;
__global__ __launch_bounds__(kBlock) void ds_time_rank_kernel(
    const int* __restrict__ val, long long n, const int* __restrict__ start,
    const int* __restrict__ cells, const float* __restrict__ t, int* __restrict__ order,
    int* __restrict__ unranked, BuildReport* __restrict__ report) {
  __shared__ float ts[kRankChunk];
  __shared__ int first, last;
  const int C = *cells;
  for (long long b0 = (long long)blockIdx.x * kBlock; b0 < n; b0 += (long long)gridDim.x * kBlock) {
    const int i = (int)min(b0 + threadIdx.x, n - 1);
    int lo = 0, hi = C;  // start[lo] <= i < start[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (start[mid] <= i) lo = mid; else hi = mid;
    }
    const int s = start[lo], e = start[lo + 1];
    const bool live = b0 + threadIdx.x < n, deep = e - s > kMaxRanked;
    if (deep) {
      *unranked = 1;
      report->deep = 1;
    }
    const int me = val[i];
    const float ti = t[me];
    if (threadIdx.x == 0) {
      first = INT_MAX;
      last = 0;
    }
    __syncthreads();
    if (!deep) {
      atomicMin(&first, s);
      atomicMax(&last, e);
    }
    __syncthreads();
    const int from = first, to = last;
    int rank = 0;
    for (int c0 = from; c0 < to; c0 += kRankChunk) {
      __syncthreads();  // the chunk before (and the bounds) have been read
#pragma unroll
      for (int q = 0; q < kRankChunk / kBlock; ++q) {
        const int j = c0 + q * kBlock + threadIdx.x;
        ts[q * kBlock + threadIdx.x] = t[val[min(j, to - 1)]];
      }
      __syncthreads();
      // positions within a cell are in index order
      const int a = max(s, c0), b = deep ? a : min(e, c0 + kRankChunk);
#pragma unroll 8
      for (int j = a; j < b; ++j) {
        const float tj = ts[j - c0];
        rank += (int)(tj < ti) | ((int)(tj == ti) & (int)(j < i));
      }
    }
    if (live && !deep) order[s + rank] = me;
    __syncthreads();
  }
}

// Which threads the cells of a walk go to: a walk is a chain of dependent loads per cell, and a wave
// takes as long as all its lanes' gathers together, so cells of many points get waves of their own: every
// (1 << s)-th thread has one, as many apart as n allows. Packed into the first threads, 260,000 points in
// cells of 1,024 took 1,449 us to write (now 554), the whole filter 2,414 (now 1,134); two or four times
// denser than this cost 53,000 points in cells of 64 up to 13 % and gained 260,000 in cells of 128 up to 8 %.
__device__ inline int walk_shift(long long n, int cells) {
  int s = 0;
  while (s < 6 && ((long long)cells << (s + 1)) <= n) ++s;
  return s;
}

// One thread per cell walks the cell's points in (time, index) order: the count pass stores the
// number of its voxels (0 past the cells), the emit pass writes every voxel's means at the offsets
// of the scanned counts, unless they exceed the capacity.
template <bool EMIT>
__global__ __launch_bounds__(kBlock) void ds_walk_kernel(
    const int* __restrict__ val, long long n, const int* __restrict__ start,
    const int* __restrict__ cells, const int* __restrict__ unranked,
    const float* __restrict__ xyz, const float* __restrict__ t, double thr,
    int* __restrict__ vcount, const int* __restrict__ voff, const int* __restrict__ total,
    long long capacity, float* __restrict__ out, float* __restrict__ tout,
    BuildReport* __restrict__ report) {
#pragma clang fp contract(off)
  if (unranked && *unranked) return;  // a cell has no order yet: the call starts again by time
  const int C = *cells;
  const long long m = EMIT ? *total : 0;
  if (EMIT && blockIdx.x == 0 && threadIdx.x == 0) report->count = (int)m;
  if (EMIT && m > capacity) return;
  const int shift = walk_shift(n, C);  // C << shift <= n
  for (long long at = (long long)blockIdx.x * blockDim.x + threadIdx.x; at < n;
       at += (long long)gridDim.x * blockDim.x) {
    if (!EMIT && at >= C) vcount[at] = 0;
    const long long i = at >> shift;
    if (i >= C || (i << shift) != at) continue;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, st = 0.0;
    int cnt = 0, nv = 0;
    const long long o = EMIT ? voff[i] : 0;
    const int e = start[i + 1];
    for (int j = start[i]; j < e; ++j) {
      const long long p = val[j];
      const double tj = t ? (double)t[p] : 0.0;
      if (t && cnt > 0 && fabs(tj - st / (double)cnt) > thr) {
        if (EMIT && o + nv < m) {
          out[o + nv] = (float)(s0 / (double)cnt);
          out[m + o + nv] = (float)(s1 / (double)cnt);
          out[2 * m + o + nv] = (float)(s2 / (double)cnt);
          if (tout) tout[o + nv] = (float)(st / (double)cnt);
        }
        ++nv;
        s0 = s1 = s2 = st = 0.0;
        cnt = 0;
      }
      if (EMIT) {
        s0 = s0 + (double)xyz[p];
        s1 = s1 + (double)xyz[n + p];
        s2 = s2 + (double)xyz[2 * n + p];
      }
      st = st + tj;
      ++cnt;
    }
    if (EMIT && o + nv < m) {
      out[o + nv] = (float)(s0 / (double)cnt);
      out[m + o + nv] = (float)(s1 / (double)cnt);
      out[2 * m + o + nv] = (float)(s2 / (double)cnt);
      if (tout) tout[o + nv] = (float)(st / (double)cnt);
    }
    ++nv;
    if (!EMIT) vcount[i] = nv;
  }
}

// ------------------------------------------------------------------ k nearest neighbours

struct CellSlot {
  unsigned long long key;  // Morton code of the cell, kEmptyCell if free
  int start, count;        // the cell's points in the sorted cloud
};

__device__ inline unsigned long long morton3(int x, int y, int z) {
  return spread3((unsigned)x) | (spread3((unsigned)y) << 1) | (spread3((unsigned)z) << 2);
}

__device__ inline unsigned cell_hash(unsigned long long k) {  // SplitMix64 finalizer
  k ^= k >> 30;
  k *= 0xbf58476d1ce4e5b9ull;
  k ^= k >> 27;
  k *= 0x94d049bb133111ebull;
  k ^= k >> 31;
  return (unsigned)k;
}

// A float's bits as an int in the floats' order (its own inverse).
__host__ __device__ inline int ordered_bits(int b) { return b ^ ((b >> 31) & 0x7fffffff); }

// Minimum and maximum of every axis (as ordered bits), and the finiteness check.
__global__ __launch_bounds__(kBlock) void knn_bounds_kernel(const float* __restrict__ xyz,
                                                            long long n, int* __restrict__ bounds,
                                                            BuildReport* __restrict__ report) {
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
  bool bad = false;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    for (int a = 0; a < 3; ++a) {
      const float v = xyz[a * n + i];
      bad |= !isfinite(v);
      const int b = ordered_bits(__float_as_int(v));
      lo[a] = min(lo[a], b);
      hi[a] = max(hi[a], b);
    }
  publish_bounds(lo, hi, bounds, report);
  if (bad) report->nonfinite = 1;
}

// Cell size estimate: for S sampled points (one block each), the binary exponent e of the
// squared distance at which the count of points reaches k; the k-th neighbour then lies within
// 2^((e + 1) / 2). est = INT_MAX if the cloud has fewer than k points, INT_MIN for duplicates.
// Most distances share a few exponents, so every lane of 16 counts in a copy of its own (one copy
// for all lanes serialized on them: 31 us for 19,000 points); four points' loads are in flight per lane
// (one: 20 us, four: 12.6).
constexpr int kExpBins = 128, kExpCopies = 16, kSampleBlock = 512;
__global__ __launch_bounds__(kSampleBlock) void knn_sample_kernel(const float* __restrict__ xyz,
                                                                  long long n, int S, int k,
                                                                  BuildReport* __restrict__ report) {
#pragma clang fp contract(off)
  __shared__ int hist[kExpBins][kExpCopies + 1];
  for (int b = threadIdx.x; b < kExpBins * (kExpCopies + 1); b += blockDim.x) (&hist[0][0])[b] = 0;
  __syncthreads();
  const long long q = (long long)blockIdx.x * n / S;
  const double q0 = xyz[q], q1 = xyz[n + q], q2 = xyz[2 * n + q];
  constexpr int kAhead = 4;
  for (long long j0 = threadIdx.x; j0 < n; j0 += (long long)kAhead * kSampleBlock) {
    float x[kAhead], y[kAhead], z[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const long long j = min(j0 + (long long)u * kSampleBlock, n - 1);
      x[u] = xyz[j];
      y[u] = xyz[n + j];
      z[u] = xyz[2 * n + j];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (j0 + (long long)u * kSampleBlock >= n) break;
      const double dx = (double)x[u] - q0, dy = (double)y[u] - q1, dz = (double)z[u] - q2;
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      const int b = d2 > 0.0 ? min(max(ilogb(d2), -62), 62) + 64 : 0;
      atomicAdd(&hist[b][threadIdx.x & (kExpCopies - 1)], 1);
    }
  }
  __syncthreads();
  if (threadIdx.x < kExpBins) {
    int c = 0;
    for (int r = 0; r < kExpCopies; ++r) c += hist[threadIdx.x][r];
    hist[threadIdx.x][kExpCopies] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int cum = 0, e = INT_MAX;
    for (int b = 0; b < kExpBins; ++b) {
      cum += hist[b][kExpCopies];
      if (cum >= k) {
        e = b == 0 ? INT_MIN : b - 64;
        break;
      }
    }
    report->est[blockIdx.x] = e;
  }
}

// Morton code of every point's cell (coordinates relative to the cloud's lowest cell). One block per
// sort tile; hist (may be null): the first pass's digit counts.
__global__ __launch_bounds__(kBlock) void knn_code_kernel(const float* __restrict__ xyz,
                                                          long long n, double inv_h, int lx,
                                                          int ly, int lz,
                                                          unsigned long long* __restrict__ code,
                                                          int* __restrict__ idx,
                                                          int* __restrict__ hist) {
  unsigned digit[kSortTile / kBlock];
  bool valid[kSortTile / kBlock];
#pragma unroll
  for (int q = 0; q < kSortTile / kBlock; ++q) {
    const long long i = (long long)blockIdx.x * kSortTile + q * kBlock + threadIdx.x;
    valid[q] = i < n;
    digit[q] = 0;
    if (!valid[q]) continue;
    const int cx = (int)floor((double)xyz[i] * inv_h) - lx;
    const int cy = (int)floor((double)xyz[n + i] * inv_h) - ly;
    const int cz = (int)floor((double)xyz[2 * n + i] * inv_h) - lz;
    const unsigned long long c = morton3(cx, cy, cz);
    code[i] = c;
    idx[i] = (int)i;
    digit[q] = (unsigned)c;
  }
  if (hist) sort_tile_hist(digit, valid, hist + (size_t)blockIdx.x * 256);
}

// Sorted copy of the positions, each with its point's index (one 16-byte load per candidate).
struct alignas(16) SortedPoint {
  float x, y, z;
  int id;
};
__global__ __launch_bounds__(kBlock) void knn_gather_kernel(const float* __restrict__ xyz,
                                                            long long n,
                                                            const int* __restrict__ perm,
                                                            SortedPoint* __restrict__ xs) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int p = perm[i];
    xs[i] = SortedPoint{xyz[p], xyz[n + p], xyz[2 * n + p], p};
  }
}

// Grid level L has cells 8^L times the finest along each axis; its cell of a point is the
// finest cell's relative coordinates shifted right by 3L, so its Morton code is the finest code
// shifted right by 9L and every level's cells are contiguous runs of the one sorted order.
// Two launches for all levels (blockIdx.y): a cell's first position claims a hash slot and stores its
// start, then its last position finds the slot and stores the count.
constexpr int kMaxLevels = 8;  // 3 more bits per level: 8 levels cover 2^21 finest cells
struct LevelTables {
  CellSlot* slots[kMaxLevels];
  unsigned mask[kMaxLevels];
};

__global__ __launch_bounds__(kBlock) void knn_level_head_kernel(
    long long n, const unsigned long long* __restrict__ code, LevelTables tab,
    int* __restrict__ internal) {
  const int shift = 9 * blockIdx.y;
  CellSlot* slots = tab.slots[blockIdx.y];
  const unsigned mask = tab.mask[blockIdx.y];
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const unsigned long long c = code[i] >> shift;
    if (i > 0 && (code[i - 1] >> shift) == c) continue;
    unsigned s = cell_hash(c) & mask;
    bool placed = false;
    for (unsigned probe = 0; probe <= mask; ++probe) {
      const unsigned long long prev = atomicCAS(&slots[s].key, kEmptyCell, c);
      if (prev == kEmptyCell) {
        slots[s].start = (int)i;
        placed = true;
        break;
      }
      s = (s + 1) & mask;
    }
    if (!placed) *internal = 1;
  }
}

__global__ __launch_bounds__(kBlock) void knn_level_tail_kernel(
    long long n, const unsigned long long* __restrict__ code, LevelTables tab,
    int* __restrict__ internal) {
  const int shift = 9 * blockIdx.y;
  CellSlot* slots = tab.slots[blockIdx.y];
  const unsigned mask = tab.mask[blockIdx.y];
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const unsigned long long c = code[i] >> shift;
    if (i + 1 < n && (code[i + 1] >> shift) == c) continue;
    unsigned s = cell_hash(c) & mask;
    bool found = false;
    for (unsigned probe = 0; probe <= mask; ++probe) {
      if (slots[s].key == c) {
        slots[s].count = (int)(i + 1 - slots[s].start);
        found = true;
        break;
      }
      s = (s + 1) & mask;
    }
    if (!found) *internal = 1;
  }
}

struct KnnGrid {
  const SortedPoint* xs;   // [n] sorted positions and original indices
  const CellSlot* slots[kMaxLevels];
  unsigned mask[kMaxLevels];
  int levels;
  double h, inv_h;         // finest cell edge (a power of two) and its inverse
  int lo[3];               // lowest finest cell per axis
  int ext[3];              // highest relative finest cell per axis
  long long n;
};

__device__ inline const CellSlot* find_cell(const CellSlot* slots, unsigned mask,
                                            unsigned long long c) {
  unsigned s = cell_hash(c) & mask;
  for (unsigned probe = 0; probe <= mask; ++probe) {
    const unsigned long long k = slots[s].key;
    if (k == c) return &slots[s];
    if (k == kEmptyCell) return nullptr;
    s = (s + 1) & mask;
  }
  return nullptr;
}

// Offers candidate (d, id) to the k best pairs kept sorted in bd/bi (K >= k slots): a better
// candidate bubbles down with selects; kth/kthi track slot k - 1.
template <int K>
__device__ inline void offer(double d, int id, double (&bd)[K], int (&bi)[K], double& kth,
                             int& kthi, int k) {
  if (!(d < kth || (d == kth && id < kthi))) return;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const bool lt = d < bd[s] || (d == bd[s] && id < bi[s]);
    const double td = bd[s];
    const int ti = bi[s];
    bd[s] = lt ? d : td;
    bi[s] = lt ? id : ti;
    d = lt ? td : d;
    id = lt ? ti : id;
  }
  kth = bd[0];
  kthi = bi[0];
#pragma unroll
  for (int s = 1; s < K; ++s)
    if (s == k - 1) {
      kth = bd[s];
      kthi = bi[s];
    }
}

// Shells searched on one level before the search moves to the next, coarser one.
constexpr int kMaxShell = 3;
// Lanes that share one query.
constexpr int kGroup = 16;

// Rotation and upward shift (zeros enter) within the 16 lanes of a row: register moves, where a
// shuffle goes through LDS.
template <int N>
__device__ inline int row_ror(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false);
}
template <int N>
__device__ inline int row_shr0(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x110 + N, 0xf, 0xf, true);
}
template <int N>
__device__ inline void row_least(double& d, int& id) {
  const double od = __hiloint2double(row_ror<N>(__double2hiint(d)), row_ror<N>(__double2loint(d)));
  const int oi = row_ror<N>(id);
  const bool lt = od < d || (od == d && oi < id);
  d = lt ? od : d;
  id = lt ? oi : id;
}

// The group's `rounds` best pairs in order: every lane offers the head of its own sorted list,
// rotations over the group's lanes find the least (distance, index), its owner advances.
// Returns the pair of the last round (the group's k-th); `out`, if given, receives round s at
// out[s * n] from lane s mod kGroup.
template <int K>
__device__ inline void group_select(const double (&bd)[K], const int (&bi)[K], int rounds,
                                    int lane, double& kd, int& ki, int* out, long long n) {
  int head = 0;
  for (int s = 0; s < rounds; ++s) {
    double hd = INFINITY;
    int hi = INT_MAX;
#pragma unroll
    for (int t = 0; t < K; ++t)
      if (t == head) {
        hd = bd[t];
        hi = bi[t];
      }
    double md = hd;
    int mi = hi;
    row_least<8>(md, mi);
    row_least<4>(md, mi);
    row_least<2>(md, mi);
    row_least<1>(md, mi);
    if (mi != INT_MAX && mi == hi) ++head;  // indices are unique: exactly one owner
    if (out && (s % kGroup) == lane) out[(long long)s * n] = mi == INT_MAX ? -1 : mi;
    kd = md;
    ki = mi;
  }
}

// kGroup lanes per query, queries in sorted order (neighbouring groups query neighbouring
// points). On level L the search grows cubes of level-L cells around the query's cell: first
// the 3 x 3 x 3 cube, then the shells at Chebyshev distance 2, 3, ...; the lanes look up the
// cells of a step kGroup at a time, one each, and then share out the points of those cells
// (every lane takes every kGroup-th point, so the few large cells of an isolated query's coarse
// levels are split too); each lane keeps the best pairs it has seen sorted in registers
// (K >= k slots; a better candidate bubbles down with selects). After
// every step the group's k-th pair is merged from the lanes' lists. Every unvisited point lies
// outside the searched cube, at least `bound` away, so the search ends once the k-th distance is
// below bound^2 (with a relative margin far above the rounding of either side). A query still open
// after shell kMaxShell moves one level up: there the first 3 x 3 x 3 cube covers the previous
// level's cube (kMaxShell < 8), whose points were visited already and are skipped. The top level
// is one cell, so every query ends.
template <int K>
__global__ __launch_bounds__(kBlock) void knn_query_kernel(KnnGrid g, int k,
                                                           int* __restrict__ nbr) {
#pragma clang fp contract(off)
  const long long n = g.n;
  const int lane = threadIdx.x & (kGroup - 1);
  const long long stride = (long long)gridDim.x * blockDim.x / kGroup;
  for (long long i = ((long long)blockIdx.x * blockDim.x + threadIdx.x) / kGroup; i < n;
       i += stride) {
    const SortedPoint me = g.xs[i];
    const double q0 = me.x, q1 = me.y, q2 = me.z;
    const int f0 = (int)floor(q0 * g.inv_h) - g.lo[0];
    const int f1 = (int)floor(q1 * g.inv_h) - g.lo[1];
    const int f2 = (int)floor(q2 * g.inv_h) - g.lo[2];
    double bd[K];
    int bi[K];
#pragma unroll
    for (int s = 0; s < K; ++s) {
      bd[s] = INFINITY;
      bi[s] = INT_MAX;
    }
    double kth = INFINITY;  // this lane's k-th
    int kthi = INT_MAX;
    double gk = INFINITY;   // the group's k-th (equal in all its lanes)
    int gki = INT_MAX;
    const double o0 = (double)g.lo[0] * g.h, o1 = (double)g.lo[1] * g.h,
                 o2 = (double)g.lo[2] * g.h;
    bool done = false;
    for (int L = 0; L < g.levels && !done; ++L) {
      const int sh = 3 * L;
      const double hl = g.h * (double)(1 << sh);
      const int c0 = f0 >> sh, c1 = f1 >> sh, c2 = f2 >> sh;
      const int x1 = g.ext[0] >> sh, y1 = g.ext[1] >> sh, z1 = g.ext[2] >> sh;
      const int psh = sh - 3;  // previous level's cells (L > 0)
      const int p0 = L > 0 ? f0 >> psh : 0, p1 = L > 0 ? f1 >> psh : 0,
                p2 = L > 0 ? f2 >> psh : 0;
      const CellSlot* slots = g.slots[L];
      const unsigned mask = g.mask[L];
      for (int r = 1; r <= kMaxShell; ++r) {
        const bool first = r == 1;  // the whole 3 x 3 x 3 cube
        const bool skip_seen = L > 0 && first;
        // the step's cells, indexed over the cube of side 2r + 1 (the interior of a shell is
        // skipped): each lane looks up one cell per round, then the group walks the points of
        // the round's cells together, every lane taking every kGroup-th point
        const int side = 2 * r + 1, ncube = side * side * side;
        for (int base = 0; base < ncube; base += kGroup) {
          int start = 0, count = 0;
          const int t = base + lane;
          if (t < ncube) {
            const int dx = t % side - r, dy = (t / side) % side - r, dz = t / (side * side) - r;
            const int x = c0 + dx, y = c1 + dy, z = c2 + dz;
            const bool in_step = first || abs(dx) == r || abs(dy) == r || abs(dz) == r;
            bool want = in_step && x >= 0 && x <= x1 && y >= 0 && y <= y1 && z >= 0 && z <= z1;
            if (want && gk < INFINITY) {  // skip cells that cannot hold a better point
              const double b0 = o0 + (double)x * hl, b1 = o1 + (double)y * hl,
                           b2 = o2 + (double)z * hl;
              const double e0 = q0 < b0 ? b0 - q0 : (q0 > b0 + hl ? q0 - (b0 + hl) : 0.0);
              const double e1 = q1 < b1 ? b1 - q1 : (q1 > b1 + hl ? q1 - (b1 + hl) : 0.0);
              const double e2 = q2 < b2 ? b2 - q2 : (q2 > b2 + hl ? q2 - (b2 + hl) : 0.0);
              want = ((e0 * e0 + e1 * e1) + e2 * e2) * (1.0 - 1e-12) <= gk;
            }
            if (want) {
              const CellSlot* cs = find_cell(slots, mask, morton3(x, y, z));
              if (cs) {
                start = cs->start;
                count = cs->count;
              }
            }
          }
          // the cells' points as one list: lane l takes its entries l, l + 16, ... (two in flight)
          int inc = count;
          inc += row_shr0<1>(inc);
          inc += row_shr0<2>(inc);
          inc += row_shr0<4>(inc);
          inc += row_shr0<8>(inc);
          const int total = __shfl(inc, kGroup - 1, kGroup), excl = inc - count;
          const int shift0 = start - excl;  // position of the list's entry c in this lane's cell: c + shift0
          for (int c0 = 0; c0 < total; c0 += 2 * kGroup) {
            SortedPoint p[2];
            bool have[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int c = c0 + h * kGroup + lane;
              int cell = 0;  // the last cell whose entries begin at or before c
#pragma unroll
              for (int step = kGroup / 2; step > 0; step >>= 1)
                if (__shfl(excl, cell + step, kGroup) <= c) cell += step;
              const int j = c + __shfl(shift0, cell, kGroup);
              have[h] = c < total;
              p[h] = g.xs[have[h] ? j : i];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              if (!have[h]) continue;
              const double x0 = p[h].x, x1_ = p[h].y, x2 = p[h].z;
              if (skip_seen) {
                const int d0 = (((int)floor(x0 * g.inv_h) - g.lo[0]) >> psh) - p0;
                const int d1 = (((int)floor(x1_ * g.inv_h) - g.lo[1]) >> psh) - p1;
                const int d2 = (((int)floor(x2 * g.inv_h) - g.lo[2]) >> psh) - p2;
                if (abs(d0) <= kMaxShell && abs(d1) <= kMaxShell && abs(d2) <= kMaxShell)
                  continue;  // visited on the previous level
              }
              const double dx_ = x0 - q0, dy_ = x1_ - q1, dz_ = x2 - q2;
              const double d = (dx_ * dx_ + dy_ * dy_) + dz_ * dz_;
              const int id = p[h].id;
              if (d > gk || (d == gk && id > gki)) continue;  // cannot reach the group's k
              offer<K>(d, id, bd, bi, kth, kthi, k);
            }
          }
        }
        group_select<K>(bd, bi, k, lane, gk, gki, nullptr, n);
        if (c0 - r <= 0 && c1 - r <= 0 && c2 - r <= 0 && c0 + r >= x1 && c1 + r >= y1 &&
            c2 + r >= z1) {
          done = true;  // every cell visited
          break;
        }
        const double g0 = fmin(q0 - (o0 + (double)(c0 - r) * hl), o0 + (double)(c0 + r + 1) * hl - q0);
        const double g1 = fmin(q1 - (o1 + (double)(c1 - r) * hl), o1 + (double)(c1 + r + 1) * hl - q1);
        const double g2 = fmin(q2 - (o2 + (double)(c2 - r) * hl), o2 + (double)(c2 + r + 1) * hl - q2);
        const double bound = fmax(fmin(fmin(g0, g1), g2), 0.0);
        if (gk < bound * bound * (1.0 - 1e-12)) {
          done = true;
          break;
        }
      }
    }
    group_select<K>(bd, bi, k, lane, gk, gki, nbr + me.id, n);
  }
}

// ------------------------------------------------------------------ point covariances

// Cyclic Jacobi iteration on a symmetric 3x3 A (Golub & Van Loan, symmetric Schur rotations):
// A -> V^T A V diagonal, V orthogonal.
__device__ inline void rotate(double (&A)[3][3], double (&V)[3][3], int p, int q) {
  if (A[p][q] == 0.0) return;
  const double theta = (A[q][q] - A[p][p]) / (2.0 * A[p][q]);
  const double at = fabs(theta);
  const double t = at > 1e150 ? 0.5 / theta
                              : (theta >= 0.0 ? 1.0 : -1.0) / (at + sqrt(at * at + 1.0));
  const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const double arp = A[r][p], arq = A[r][q];
    A[r][p] = c * arp - s * arq;
    A[r][q] = s * arp + c * arq;
  }
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const double apr = A[p][r], aqr = A[q][r];
    A[p][r] = c * apr - s * aqr;
    A[q][r] = s * apr + c * aqr;
  }
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const double vrp = V[r][p], vrq = V[r][q];
    V[r][p] = c * vrp - s * vrq;
    V[r][q] = s * vrp + c * vrq;
  }
}

// Neighbours s .. s + kCovAhead - 1 of point i, their loads in flight together (one neighbour at a time
// the loop waited twice for memory for each: 19.2 us for 18,000 points of 10, now 17.8, most of it the
// rotations); returns which of them exist, bad: an index past the cloud.
constexpr int kCovAhead = 5;
__device__ inline unsigned cov_neighbors(const float* __restrict__ xyz, long long n,
                                         const int* __restrict__ nbr, int k, int s, long long i,
                                         float (&p)[kCovAhead][3], bool& bad) {
  int j[kCovAhead];
#pragma unroll
  for (int u = 0; u < kCovAhead; ++u) j[u] = s + u < k ? nbr[(s + u) * n + i] : -1;
  unsigned ok = 0;
#pragma unroll
  for (int u = 0; u < kCovAhead; ++u) {
    bad |= j[u] >= n;
    const bool in = j[u] >= 0 && j[u] < n;
    ok |= in ? 1u << u : 0u;
    const long long q = in ? j[u] : i;
    p[u][0] = xyz[q];
    p[u][1] = xyz[n + q];
    p[u][2] = xyz[2 * n + q];
  }
  return ok;
}

__global__ __launch_bounds__(kBlock) void cov_kernel(const float* __restrict__ xyz, long long n,
                                                     const int* __restrict__ nbr, int k,
                                                     double scale, double eps,
                                                     float* __restrict__ cov,
                                                     unsigned* __restrict__ flags) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    double m0 = 0.0, m1 = 0.0, m2 = 0.0;
    int m = 0;
    bool bad = false;
    for (int s = 0; s < k; s += kCovAhead) {
      float p[kCovAhead][3];
      const unsigned ok = cov_neighbors(xyz, n, nbr, k, s, i, p, bad);
#pragma unroll
      for (int u = 0; u < kCovAhead; ++u) {
        if (!(ok >> u & 1u)) continue;
        m0 += (double)p[u][0];
        m1 += (double)p[u][1];
        m2 += (double)p[u][2];
        ++m;
      }
    }
    if (bad) atomicOr(flags, kFlagBadIndex);
    const double inv_m = m > 0 ? 1.0 / (double)m : 0.0;
    m0 *= inv_m;
    m1 *= inv_m;
    m2 *= inv_m;
    double A[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    for (int s = 0; s < k; s += kCovAhead) {
      float p[kCovAhead][3];
      const unsigned ok = cov_neighbors(xyz, n, nbr, k, s, i, p, bad);
#pragma unroll
      for (int u = 0; u < kCovAhead; ++u) {
        if (!(ok >> u & 1u)) continue;
        const double v[3] = {(double)p[u][0] - m0, (double)p[u][1] - m1, (double)p[u][2] - m2};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int b = a; b < 3; ++b) A[a][b] += v[a] * v[b];
      }
    }
    A[1][0] = A[0][1];
    A[2][0] = A[0][2];
    A[2][1] = A[1][2];
    double c6[6];
    if (scale > 0.0) {
      double V[3][3] = {{1.0, 0.0, 0.0}, {0.0, 1.0, 0.0}, {0.0, 0.0, 1.0}};
      for (int sweep = 0; sweep < 12; ++sweep) {
        const double off = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
        const double dia = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2];
        if (off <= 1e-36 * dia) break;
        rotate(A, V, 0, 1);
        rotate(A, V, 0, 2);
        rotate(A, V, 1, 2);
      }
      int c = 0;
      if (A[1][1] < A[c][c]) c = 1;
      if (A[2][2] < A[c][c]) c = 2;
      const double u[3] = {c == 0 ? V[0][0] : (c == 1 ? V[0][1] : V[0][2]),
                           c == 0 ? V[1][0] : (c == 1 ? V[1][1] : V[1][2]),
                           c == 0 ? V[2][0] : (c == 1 ? V[2][1] : V[2][2])};
      const double g = 1.0 - eps;
      c6[0] = scale * (1.0 - g * u[0] * u[0]);
      c6[1] = scale * (-g * u[0] * u[1]);
      c6[2] = scale * (-g * u[0] * u[2]);
      c6[3] = scale * (1.0 - g * u[1] * u[1]);
      c6[4] = scale * (-g * u[1] * u[2]);
      c6[5] = scale * (1.0 - g * u[2] * u[2]);
    } else {
      c6[0] = A[0][0] * inv_m;
      c6[1] = A[0][1] * inv_m;
      c6[2] = A[0][2] * inv_m;
      c6[3] = A[1][1] * inv_m;
      c6[4] = A[1][2] * inv_m;
      c6[5] = A[2][2] * inv_m;
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) cov[a * n + i] = (float)c6[a];
  }
}

bool pow2_res(double res) {
  int e = 0;
  return std::frexp(res, &e) == 0.5;
}

}  // namespace

vgicp_status downsample(const float* xyz, const float* t, int64_t n, double res, double d_scan,
                        float* xyz_out, float* t_out, int64_t capacity, int64_t* n_out,
                        hipStream_t s) {
  *n_out = 0;
  if (n == 0) return VGICP_OK;
  HostBlock hb;
  if (!hb.p) return fail(VGICP_E_OOM, "pinned host block");
  BuildReport* report = static_cast<BuildReport*>(hb.p);
  volatile BuildReport* rep = report;
  const bool small = n <= kSortMax;
  const size_t words = small ? sort_hist_ints(1, n) : 0, N = (size_t)n;
  Arena ar(&hb);
  ar.need<int>(3 * N);
  ar.need<int>(8);
  ar.need<int>(words);
  ar.need<unsigned long long>(N);
  ar.need<unsigned long long>(N);
  for (int i = 0; i < 5; ++i) ar.need<int>(N);
  ar.need<int>(N + 1);
  ar.need<int>(kRunTiles);
  ar.need<int>(3);
  hipError_t e;
  if ((e = ar.get(s))) return hip_fail(e, "device block (downsample)");
  int* kc = ar.take<int>(3 * N);
  int* bounds = ar.take<int>(8);
  SortBuffers sb;
  sb.hist = ar.take<int>(words);
  sb.k = ar.take<unsigned long long>(N);
  sb.kt = ar.take<unsigned long long>(N);
  sb.v = ar.take<int>(N);
  sb.vt = ar.take<int>(N);
  int* vcnt = ar.take<int>(N);
  int* voff = ar.take<int>(N);
  int* ranked = ar.take<int>(N);
  int* start = ar.take<int>(N + 1);
  int* tile_counts = ar.take<int>(kRunTiles);
  int* totals = ar.take<int>(3);  // cells, voxels, a cell left unranked
  const bool p2 = pow2_res(res);
  launch_call_init(&totals[2], 1, bounds, report, s);
  ds_cells_kernel<<<std::min(grid_for(n), 128), kBlock, 0, s>>>(xyz, t, n, p2 ? 1 : 0, res, 1.0 / res, kc,
                                                 bounds, report);
  if ((e = hipGetLastError()) || (e = hipStreamSynchronize(s)))
    return hip_fail(e, "downsample cells");
  if (rep->nonfinite) return fail(VGICP_E_NONFINITE, "non-finite point or timestamp");
  if (rep->keyrange) return fail(VGICP_E_KEY_RANGE, "cell coordinate out of range");
  const int lo[3] = {rep->lo[0], rep->lo[1], rep->lo[2]};
  const int bx = bits_for((long long)rep->hi[0] - lo[0]), by = bits_for((long long)rep->hi[1] - lo[1]),
            bz = bits_for((long long)rep->hi[2] - lo[2]);
  const double thr = d_scan / 10.0;
  // the cells' points in (time, index) order: sorted by cell and ranked within the cells, or (long
  // clouds, or a cell too full to rank) sorted by time first, which the stable cell sort keeps
  bool by_time = t != nullptr && !small;
  for (;;) {
    Scratch sc;
    const int* order = nullptr;
    auto sort = [&](int bits) {
      return small ? sort_passes(sb, nullptr, 1, n, bits, &report->internal, s)
                   : radix_sort_pairs(&sb.k, &sb.v, &sb.kt, &sb.vt, n, bits, &report->internal, s, sc);
    };
    int* hist = small ? sb.hist : nullptr;
    if (by_time) {
      ds_time_key_kernel<<<(unsigned)sort_tiles(n), kBlock, 0, s>>>(t, n, sb.k, sb.v, hist);
      if ((e = hipGetLastError()) || (e = sort(32))) return hip_fail(e, "downsample time sort");
      order = sb.v;
    }
    ds_cell_key_kernel<<<(unsigned)sort_tiles(n), kBlock, 0, s>>>(
        kc, n, order, lo[0], lo[1], lo[2], by + bz, bz, sb.kt, sb.vt, hist);
    std::swap(sb.k, sb.kt);
    std::swap(sb.v, sb.vt);
    if ((e = sort(bx + by + bz))) return hip_fail(e, "downsample cell sort");
    if ((e = run_starts(sb.k, n, start, tile_counts, &totals[0], s)))
      return hip_fail(e, "downsample cells");
    const int* val = sb.v;
    int* unranked = nullptr;
    if (t && !by_time) {
      unranked = &totals[2];
      ds_time_rank_kernel<<<grid_for(n), kBlock, 0, s>>>(sb.v, n, start, &totals[0], t, ranked,
                                                         unranked, report);
      val = ranked;
    }
    ds_walk_kernel<false><<<grid_for(n), kBlock, 0, s>>>(
        val, n, start, &totals[0], unranked, xyz, t, thr, vcnt, nullptr, nullptr, 0, nullptr, nullptr,
        report);
    if ((e = hipGetLastError()) || (e = scan_values(vcnt, voff, n, tile_counts, &totals[1], s)))
      return hip_fail(e, "downsample count");
    ds_walk_kernel<true><<<grid_for(n), kBlock, 0, s>>>(val, n, start, &totals[0], unranked, xyz, t,
                                                        thr, nullptr, voff, &totals[1], capacity,
                                                        xyz_out, t ? t_out : nullptr, report);
    if ((e = hipGetLastError()) || (e = hipStreamSynchronize(s)))
      return hip_fail(e, "downsample emit");
    if (!rep->deep || by_time) break;
    by_time = true;  // a cell has no order: the walks have counted and written nothing
  }
  if (rep->internal) return fail(VGICP_E_HIP, "internal error in the downsample sort");
  const int64_t m = rep->count;
  *n_out = m;
  if (m > capacity) return fail(VGICP_E_CAPACITY, "downsampled cloud exceeds the output capacity");
  return VGICP_OK;
}

vgicp_status knn(const float* xyz, int64_t n, int k, double cell, int32_t* nbr, hipStream_t s) {
  if (n == 0) return VGICP_OK;
  hipError_t e;
  HostBlock hb;
  if (!hb.p) return fail(VGICP_E_OOM, "pinned host block");
  BuildReport* report = static_cast<BuildReport*>(hb.p);
  volatile BuildReport* rep = report;
  const bool small = n <= kSortMax;
  const size_t words = small ? sort_hist_ints(1, n) : 0, N = (size_t)n;
  Arena ar(&hb);
  ar.need<int>(8);
  ar.need<int>(words);
  ar.need<unsigned long long>(N);
  ar.need<unsigned long long>(N);
  ar.need<int>(N);
  ar.need<int>(N);
  ar.need<SortedPoint>(N);
  if ((e = ar.get(s))) return hip_fail(e, "device block (knn)");
  int* bounds = ar.take<int>(8);
  SortBuffers sb;
  sb.hist = ar.take<int>(words);
  sb.k = ar.take<unsigned long long>(N);
  sb.kt = ar.take<unsigned long long>(N);
  sb.v = ar.take<int>(N);
  sb.vt = ar.take<int>(N);
  SortedPoint* xs = ar.take<SortedPoint>(N);
  launch_call_init(nullptr, 0, bounds, report, s);
  knn_bounds_kernel<<<std::min(grid_for(n), 128), kBlock, 0, s>>>(xyz, n, bounds, report);
  // the cell estimate runs beside the bounds (a non-finite cloud is rejected after it)
  const int S = cell > 0.0 ? 0 : (int)std::min<int64_t>(n, 64);
  if (S > 0) knn_sample_kernel<<<S, kSampleBlock, 0, s>>>(xyz, n, S, k, report);
  if ((e = hipGetLastError()) || (e = hipStreamSynchronize(s))) return hip_fail(e, "knn bounds");
  if (rep->nonfinite) return fail(VGICP_E_NONFINITE, "non-finite point");
  double lo[3], hi[3], maxabs = 0.0;
  for (int a = 0; a < 3; ++a) {
    const int l = ordered_bits(rep->lo[a]), h = ordered_bits(rep->hi[a]);
    float f;
    std::memcpy(&f, &l, 4);
    lo[a] = f;
    std::memcpy(&f, &h, 4);
    hi[a] = f;
    maxabs = std::max(maxabs, std::max(std::fabs(lo[a]), std::fabs(hi[a])));
  }
  int eh = 0;  // cell edge 2^eh
  if (cell > 0.0) {
    eh = (int)std::ceil(std::log2(cell));
  } else {
    std::vector<int> r;
    for (int i = 0; i < S; ++i) {
      const int v = rep->est[i];
      if (v != INT_MIN) r.push_back(v == INT_MAX ? 62 : (v + 2) / 2);  // 2^r >= k-th distance
    }
    if (!r.empty()) {
      std::nth_element(r.begin(), r.begin() + r.size() / 2, r.end());
      eh = r[r.size() / 2];
    }
  }
  // every cell coordinate stays below 2^19 in magnitude
  eh = std::max(eh, (int)std::ceil(std::log2(std::max(maxabs, 1e-300))) - 19);
  eh = std::min(std::max(eh, -60), 150);
  const double h = std::ldexp(1.0, eh), inv_h = std::ldexp(1.0, -eh);
  KnnGrid g;
  int ext_max = 0;
  for (int a = 0; a < 3; ++a) {
    g.lo[a] = (int)std::floor(lo[a] * inv_h);
    g.ext[a] = (int)std::floor(hi[a] * inv_h) - g.lo[a];
    ext_max = std::max(ext_max, g.ext[a]);
  }
  const int bits = 3 * bits_for(ext_max);
  int levels = 1;
  while (levels < kMaxLevels && (ext_max >> (3 * (levels - 1))) > 0) ++levels;
  // one buffer for the cell tables of all levels
  LevelTables tab{};
  size_t slots_total = 0, at[kMaxLevels];
  for (int L = 0; L < levels; ++L) {
    // cells on level L: at most n, and at most the product of the level's extents
    long long cells = 1;
    for (int a = 0; a < 3; ++a) cells = std::min<long long>(cells * ((g.ext[a] >> (3 * L)) + 1), n);
    unsigned cap = 1;
    while ((long long)cap < 2 * cells) cap <<= 1;
    tab.mask[L] = cap - 1;
    at[L] = slots_total;
    slots_total += cap;
  }
  Arena at_ar(&hb);
  Scratch sc;
  at_ar.need<CellSlot>(slots_total);
  if ((e = at_ar.get(s))) return hip_fail(e, "device block (knn)");
  CellSlot* slots = at_ar.take<CellSlot>(slots_total);
  for (int L = 0; L < levels; ++L) {
    tab.slots[L] = slots + at[L];
    g.slots[L] = tab.slots[L];
    g.mask[L] = tab.mask[L];
  }
  if ((e = hipMemsetAsync(slots, 0xff, slots_total * sizeof(CellSlot), s)))
    return hip_fail(e, "hipMemsetAsync");
  knn_code_kernel<<<(unsigned)sort_tiles(n), kBlock, 0, s>>>(xyz, n, inv_h, g.lo[0], g.lo[1],
                                                             g.lo[2], sb.k, sb.v,
                                                             small ? sb.hist : nullptr);
  e = small ? sort_passes(sb, nullptr, 1, n, bits, &report->internal, s)
            : radix_sort_pairs(&sb.k, &sb.v, &sb.kt, &sb.vt, n, bits, &report->internal, s, sc);
  if (e) return hip_fail(e, "knn sort");
  knn_gather_kernel<<<grid_for(n), kBlock, 0, s>>>(xyz, n, sb.v, xs);
  const dim3 lgrid((unsigned)grid_for(n), (unsigned)levels);
  knn_level_head_kernel<<<lgrid, kBlock, 0, s>>>(n, sb.k, tab, &report->internal);
  knn_level_tail_kernel<<<lgrid, kBlock, 0, s>>>(n, sb.k, tab, &report->internal);
  g.levels = levels;
  g.xs = xs;
  g.h = h;
  g.inv_h = inv_h;
  g.n = n;
  const int qgrid = grid_for(n * kGroup);
  if (k <= 6)
    knn_query_kernel<6><<<qgrid, kBlock, 0, s>>>(g, k, nbr);
  else if (k <= 10)
    knn_query_kernel<10><<<qgrid, kBlock, 0, s>>>(g, k, nbr);
  else if (k <= 16)
    knn_query_kernel<16><<<qgrid, kBlock, 0, s>>>(g, k, nbr);
  else
    knn_query_kernel<32><<<qgrid, kBlock, 0, s>>>(g, k, nbr);
  if ((e = hipGetLastError()) || (e = hipStreamSynchronize(s))) return hip_fail(e, "knn query");
  if (rep->internal) return fail(VGICP_E_HIP, "internal error in the neighbour search");
  return VGICP_OK;
}

void launch_point_covariances(const float* xyz, int64_t n, const int32_t* nbr, int k,
                              double scale, double eps, float* cov, unsigned* flags,
                              hipStream_t s) {
  if (n == 0) return;
  cov_kernel<<<grid_for(n), kBlock, 0, s>>>(xyz, n, nbr, k, scale, eps, cov, flags);
}

}  // namespace vgicp
