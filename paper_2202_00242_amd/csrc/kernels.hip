// Linearize / evaluate / backward kernels of the VGICP matching-cost factor on gfx950.
//
// Work unit: a wave's share of a tile of one factor's source points, in two phases per wave.
//   A. Lookup: every lane takes U points (structure-of-arrays loads, coalesced across the wave),
//      finds their voxels (batches: in FP32 where that is provably the FP64 voxel, in FP64 beside
//      a voxel face; single factors: in FP64), tests them against the map's bounding box and looks
//      all of them up at once. Hits are compacted into a per-wave LDS queue.
//   B. Inliers: whenever 64 are queued, all lanes take one each (covariance and voxel loads) and,
//      a row of lookups later, run the full per-point work on it (fused covariance inverse,
//      residual, 28 target-frame sums in registers). Misses thus cost only phase A.
// In a batch every wave writes its own partial sums; a single factor's block adds its waves' in order
// and writes one partial per tile. A second kernel adds the partials of each factor in (tile, wave)
// order and expands them to the factor's H and b. Results are therefore bitwise reproducible whatever
// the scheduling.
#include <algorithm>
#include <type_traits>

#include "device_math.h"
#include "internal.h"

namespace vgicp {

// ------------------------------------------------------------------ relative pose

// Row r of T_ts = T_t^-1 T_s in the fixed FP64 order of the definition (no fused multiply-add), and
// of the rounded forms used by the FP32 variants. Runs on the host (single calls) and on the
// device (batches, from the pose buffer at graph replay).
__host__ __device__ inline void rel_pose_row(const double* Tt, const double* Ts, double inv_res,
                                             int r, RelPose& o) {
#pragma clang fp contract(off)
  const double t0 = Tt[r], t1 = Tt[4 + r], t2 = Tt[8 + r];
  for (int c = 0; c < 3; ++c) {
    const double v = (t0 * Ts[c] + t1 * Ts[4 + c]) + t2 * Ts[8 + c];
    o.R[3 * r + c] = v;
    o.Rk[3 * r + c] = v * inv_res;
    o.Rf[3 * r + c] = (float)v;
    o.Rs[3 * r + c] = (float)Ts[4 * r + c];
    o.Rti[3 * r + c] = (float)Tt[4 * c + r];
  }
  const double dt[3] = {Ts[3] - Tt[3], Ts[7] - Tt[7], Ts[11] - Tt[11]};
  const double v = (t0 * dt[0] + t1 * dt[1]) + t2 * dt[2];
  o.t[r] = v;
  o.tk[r] = v * inv_res;
  o.tf[r] = (float)v;
  o.ts[r] = (float)Ts[4 * r + 3];
  o.tti[r] = (float)(-(t0 * Tt[3] + t1 * Tt[7] + t2 * Tt[11]));
}

__host__ __device__ inline void compute_rel_pose(const double* Tt, const double* Ts,
                                                 double inv_res, RelPose& o) {
  o.skip = 0;
  for (int r = 0; r < 3; ++r) rel_pose_row(Tt, Ts, inv_res, r, o);
}

void relative_pose(const double* Tt, const double* Ts, double* Tts) {
  RelPose o;
  compute_rel_pose(Tt, Ts, 1.0, o);
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c) Tts[4 * r + c] = o.R[3 * r + c];
    Tts[4 * r + 3] = o.t[r];
  }
}

RelPose make_rel_pose(const double* Tt, const double* Ts, double inv_res) {
  RelPose o;
  compute_rel_pose(Tt, Ts, inv_res, o);
  return o;
}

namespace {

// ------------------------------------------------------------------ phase A: voxel lookup

// The FP32 world-coordinate form (precision baseline): the point to world and into the target
// frame, both in FP32.
__device__ inline void naive_point(const RelPose& T, float x, float y, float z, float q[3]) {
  const float w0 = T.Rs[0] * x + T.Rs[1] * y + T.Rs[2] * z + T.ts[0];
  const float w1 = T.Rs[3] * x + T.Rs[4] * y + T.Rs[5] * z + T.ts[1];
  const float w2 = T.Rs[6] * x + T.Rs[7] * y + T.Rs[8] * z + T.ts[2];
  q[0] = T.Rti[0] * w0 + T.Rti[1] * w1 + T.Rti[2] * w2 + T.tti[0];
  q[1] = T.Rti[3] * w0 + T.Rti[4] * w1 + T.Rti[5] * w2 + T.tti[1];
  q[2] = T.Rti[6] * w0 + T.Rti[7] * w1 + T.Rti[8] * w2 + T.tti[2];
}

// Voxel coordinates of one source point in the target frame, branch-free (saturated, see
// floor_sat_i32). Returns false when the transformed point is not finite.
template <int PREC, bool DIV>
__device__ inline bool point_key(const MapView& m, const RelPose& T, float x, float y, float z,
                                 int k[3]) {
  if constexpr (PREC == kNaiveWorld) {
    float q[3];
    naive_point(T, x, y, z, q);
    const float ir = (float)m.inv_res;
    for (int a = 0; a < 3; ++a) k[a] = floor_sat_i32_f32(q[a] * ir);
    return isfinite(q[0] + q[1] + q[2]);
  } else {
    double q[3];
    if constexpr (DIV) {
      transform_exact(T.R, T.t, x, y, z, q);
      for (int a = 0; a < 3; ++a) k[a] = floor_sat_i32(q[a] / m.res);
    } else {  // q / res exactly (power-of-two res)
      transform_exact(T.Rk, T.tk, x, y, z, q);
      for (int a = 0; a < 3; ++a) k[a] = floor_sat_i32(q[a]);
    }
    return isfinite(q[0] + q[1] + q[2]);
  }
}

// Orders a wave's LDS writes before other lanes of the same wave read them.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inliers a wave may hold between batches: fewer than 64 left over plus 64 * U new ones.
template <int U>
constexpr int queue_cap() {
  return 64 * (U + 1);
}

// Buffer descriptors over the three position planes of a source cloud (n < 2^30): loads take
// a 32-bit VGPR offset against an SGPR descriptor (no per-lane 64-bit address arithmetic), and
// offsets past a plane read 0 instead of touching memory.
struct Planes {
  __amdgpu_buffer_rsrc_t x, y, z;
};

__device__ inline __amdgpu_buffer_rsrc_t raw_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                           kRawBufferFlags);
}

__device__ inline Planes make_planes(const float* xyz, int n) {
  const unsigned bytes = (unsigned)n * 4u;
  return {raw_rsrc(xyz, bytes), raw_rsrc(xyz + n, bytes), raw_rsrc(xyz + 2 * (size_t)n, bytes)};
}

// Positions of the points base + u*64 + lane, u < U. Lanes past the tile read neighbouring
// points or zeros (past the cloud), without a branch; the caller ignores them.
template <int U>
struct Chunk {
  float x[U], y[U], z[U];

  __device__ inline void load(const Planes& P, int base, int lane) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned off = (unsigned)(base + u * 64 + lane) * 4u;
      x[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(P.x, off, 0, 0));
      y[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(P.y, off, 0, 0));
      z[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(P.z, off, 0, 0));
    }
  }
};

// One queued inlier: its position (the inlier phase transforms it again in FP64: 18 operations
// for the points that hit instead of 24 more bytes of LDS for each), voxel record, point index.
struct alignas(16) QueueEntry {
  float x, y, z;
  int rec;
};
struct Queue {
  QueueEntry* e;
  int* point;
};

// Phase A of a wave-chunk: lane l resolves the points base + u*64 + l, u < U (positions in
// c), with all their lookups in flight together. Hits are appended (in (u, lane) order) to the
// wave's queue: position, voxel record index (MapView::rec) and point index; cnt
// stays wave-uniform. corr receives voxel ids.
// The next chunk's positions (nxt, at next_base) are loaded here, after this chunk's lookups
// are issued: vector-memory counters retire in issue order, so loads issued earlier would have
// to complete before the lookups could be consumed.
//
// FAST (batches): the voxel comes from an FP32 transform in voxel units relative to the map's box
// (9 FMA, RelPose::Af/sf), and is the definition's FP64 voxel whenever no coordinate lies within
// the transform's error bound of a voxel face (RelPose::thr, from the source's bounding box); a
// chunk row with a point that close (about 1 in 1,000 points at 0.5 m and 100 m) computes those
// points' voxels in FP64. VALU issue bounds this phase: the FP64 key alone is 33 of its 63
// instructions per point, the FP32 one is 20 (FP64 issues at the unpacked FP32 rate here, but the
// definition's order allows no FMA).
template <int PREC, bool DIV, int LAYOUT, int U, bool FAST, bool GRAD = false>
__device__ inline void resolve(const MapView& m, const RelPose& T, const Chunk<U>& c,
                               Chunk<U>& nxt, const Planes& P, int next_base, int base, int end,
                               int lane, const Queue& qe, int& cnt, int* __restrict__ corr,
                               unsigned& fl, float* __restrict__ gz = nullptr) {
  const float* x = c.x;
  const float* y = c.y;
  const float* z = c.z;
  unsigned slot[U], klo[U], khi[U];
  int st[U], id[U];  // st: 0 probing, 1 hit, 2 miss
#pragma unroll
  for (int u = 0; u < U; ++u) {
    id[u] = -1;
    const bool valid = base + u * 64 + lane < end;
    unsigned dx, dy, dz;  // voxel relative to the map's box
    bool inbox;
    auto exact = [&]() {
      int k[3], lo[3];
      bool finite;
      if constexpr (FAST) {
        // rare: no code of its own per key arithmetic, and no scalar registers outside this branch
        // (read ahead of the loop, its 48 words of pose and map made the loop keep its own scalars
        // in vector lanes: 22 of the 70 VALU instructions of a row; overlap rates of 160 submaps 1,481 us
        // with that, 875 without)
        const auto Tg = here(&T);
        const auto mg = here(&m);
        const bool pow2 = mg->pow2 != 0;  // point_key's two key arithmetics
        double R[9], t[3], q[3];
#pragma unroll
        for (int a = 0; a < 9; ++a) R[a] = pow2 ? Tg->Rk[a] : Tg->R[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) t[a] = pow2 ? Tg->tk[a] : Tg->t[a];
        transform_exact(R, t, x[u], y[u], z[u], q);
        finite = isfinite(q[0] + q[1] + q[2]);
        if (!pow2) {
          const double res = mg->res;
#pragma unroll
          for (int a = 0; a < 3; ++a) q[a] /= res;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) k[a] = floor_sat_i32(q[a]);
        lo[0] = mg->lo[0], lo[1] = mg->lo[1], lo[2] = mg->lo[2];
      } else {
        finite = point_key<PREC, DIV>(m, T, x[u], y[u], z[u], k);
        lo[0] = m.lo[0], lo[1] = m.lo[1], lo[2] = m.lo[2];
      }
      if (valid && !finite) fl |= kFlagNonFinite;
      dx = finite ? (unsigned)k[0] - (unsigned)lo[0] : ~0u;
      dy = (unsigned)k[1] - (unsigned)lo[1];
      dz = (unsigned)k[2] - (unsigned)lo[2];
    };
    if constexpr (FAST) {
      float s[3], f[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s[a] = fmaf(T.Af[3 * a], x[u],
                    fmaf(T.Af[3 * a + 1], y[u], fmaf(T.Af[3 * a + 2], z[u], T.sf[a])));
        f[a] = fabsf(__builtin_amdgcn_fractf(s[a]) - 0.5f);
      }
      dx = (unsigned)floor_i32_f32(s[0]);
      dy = (unsigned)floor_i32_f32(s[1]);
      dz = (unsigned)floor_i32_f32(s[2]);
      // (a cloud with a coordinate that is not finite has an infinite box: thr < 0, never sure)
      const bool sure = fmaxf(fmaxf(f[0], f[1]), f[2]) <= T.thr;
      if (__ballot(!sure) != 0ull) {
        if (!sure) exact();
      }
    } else {
      exact();
    }
    // outside the map's voxel bounding box (or out of range, or not finite): a miss
    inbox = valid && dx < (unsigned)m.ext[0] && dy < (unsigned)m.ext[1] && dz < (unsigned)m.ext[2];
    if constexpr (LAYOUT == kLayoutGrid) {
      // 24-bit multiplies: a grid has fewer than 2^24 bricks
      slot[u] = mad24(mad24(dx >> 2, (unsigned)m.gby, dy >> 2), (unsigned)m.gbz, dz >> 1);
      klo[u] = bit_in_brick_mod32(dx, dy, dz);
      khi[u] = 0;
    } else if constexpr (LAYOUT == kLayoutHash32) {
      klo[u] = (dx << (m.by + m.bz)) | (dy << m.bz) | dz;
      khi[u] = 0;
      slot[u] = hash32(klo[u]) & m.mask;
    } else {
      const long long pk = pack_key((int)dx + m.lo[0], (int)dy + m.lo[1], (int)dz + m.lo[2]);
      klo[u] = (unsigned)pk;
      khi[u] = (unsigned)((unsigned long long)pk >> 32);
      slot[u] = hash64(pk) & m.mask;
    }
    st[u] = inbox ? 0 : 2;
  }
  if constexpr (LAYOUT == kLayoutGrid) {
    // one 8-byte brick load per point, all lookahead points at once; the record position is
    // the brick's base plus the occupied voxels below the point's bit. Points outside the box
    // load past the end of the bricks, which reads an empty brick (no branch around the loads).
    const __amdgpu_buffer_rsrc_t rb = raw_rsrc(m.bricks, m.brick_bytes);
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    u32x2 br[U];  // {mask, base}, one 8-byte load each
#pragma unroll
    for (int u = 0; u < U; ++u)
      br[u] = __builtin_amdgcn_raw_buffer_load_b64(rb, st[u] == 0 ? slot[u] * 8u : 0x80000000u,
                                                   0, 0);
    nxt.load(P, next_base, lane);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned hit = __builtin_amdgcn_ubfe(br[u].x, klo[u], 1);
      id[u] = (int)br[u].y + __popc(__builtin_amdgcn_ubfe(br[u].x, 0, klo[u]));
      st[u] = hit != 0u ? 1 : 2;
    }
  } else {
    nxt.load(P, next_base, lane);
    // Linear probing, all lookahead points at once; at least three quarters of the slots are
    // free, so every probe sequence ends within capacity steps.
    for (unsigned p = 0; p <= m.mask; ++p) {
      bool pending = false;
#pragma unroll
      for (int u = 0; u < U; ++u) pending |= st[u] == 0;
      if (__ballot(pending) == 0ull) break;
      // branch-free update of every lookahead point (selects, no divergent control flow)
      if constexpr (LAYOUT == kLayoutHash32) {
        uint2 sv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) sv[u] = gbl(m.slots32)[slot[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool pend = st[u] == 0;
          const bool hit = pend && sv[u].x == klo[u];
          const bool empty = pend && sv[u].x == kEmpty32;
          id[u] = hit ? (int)sv[u].y : id[u];
          st[u] = hit ? 1 : (empty ? 2 : st[u]);
          slot[u] = (pend && !hit && !empty) ? ((slot[u] + 1) & m.mask) : slot[u];
        }
      } else {
        longlong2 sv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) sv[u] = gbl(m.slots64)[slot[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const long long key = (long long)(((unsigned long long)khi[u] << 32) | klo[u]);
          const bool pend = st[u] == 0;
          const bool hit = pend && sv[u].x == key;
          const bool empty = pend && sv[u].x == kEmpty64;
          id[u] = hit ? (int)sv[u].y : id[u];
          st[u] = hit ? 1 : (empty ? 2 : st[u]);
          slot[u] = (pend && !hit && !empty) ? ((slot[u] + 1) & m.mask) : slot[u];
        }
      }
    }
  }
  if (corr) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (base + u * 64 + lane < end) {
        int v = -1;
        if (st[u] == 1) v = (LAYOUT == kLayoutGrid) ? gbl(m.rec_id)[id[u]] : id[u];
        gblw(corr)[base + u * 64 + lane] = v;
      }
  }
  if constexpr (GRAD) {  // a point without a voxel has no gradient
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (base + u * 64 + lane < end && st[u] != 1) {
        const gptr<float> g = gblw(gz) + 3 * (size_t)(unsigned)(base + u * 64 + lane);
        g[0] = 0.0f;
        g[1] = 0.0f;
        g[2] = 0.0f;
      }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool h = st[u] == 1;
    const unsigned long long mk = __ballot(h);
    if (h) {
      const int pos = cnt + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mk >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned)mk, 0u));
      if constexpr (PREC != kCountOnly) {
        qe.e[pos] = QueueEntry{x[u], y[u], z[u], id[u]};
        qe.point[pos] = base + u * 64 + lane;
      }
    }
    cnt += __popcll(mk);
  }
}

// ------------------------------------------------------------------ phase B: inlier terms

template <int PREC>
using RealOf = typename std::conditional<PREC == kMathFp64, double, float>::type;

// One inlier with what its terms read: position, covariance, voxel record. Loaded a row of lookups
// ahead of its use (wave_body), so that the lookups cover the loads' latency.
struct Inlier {
  float x, y, z;
  int point;
  float c[6];
  double mean[3], cov[6];
};

template <bool AOS>
__device__ inline void load_inlier(const MapView& m, const float* __restrict__ cov, int n,
                                   const Queue& qe, int i, Inlier& e) {
  const QueueEntry q = qe.e[i];
  e.x = q.x;
  e.y = q.y;
  e.z = q.z;
  e.point = qe.point[i];
  if constexpr (AOS) {  // interleaved [n][6] (24 bytes): three 8-byte loads
    const gptr<const float2> c2 =
        gbl(reinterpret_cast<const float2*>(cov)) + 3 * (size_t)(unsigned)e.point;
    const float2 c01 = c2[0], c23 = c2[1], c45 = c2[2];
    e.c[0] = c01.x, e.c[1] = c01.y, e.c[2] = c23.x, e.c[3] = c23.y, e.c[4] = c45.x, e.c[5] = c45.y;
  } else {  // the caller's planes [6][n]
#pragma unroll
    for (int a = 0; a < 6; ++a) e.c[a] = gbl(cov + (size_t)a * n)[(unsigned)e.point];
  }
  const gptr<const VoxelData> v = gbl(m.rec) + (unsigned)q.rec;
#pragma unroll
  for (int a = 0; a < 3; ++a) e.mean[a] = v->mean[a];
#pragma unroll
  for (int a = 0; a < 6; ++a) e.cov[a] = v->cov[a];
}

// Full per-point work of one inlier (its voxel is known): fused covariance, inverse,
// residual and target-frame Gauss-Newton terms.
template <int PREC, bool LIN, class Acc>
__device__ inline void inlier_terms(const RelPose& T, const Inlier& e, Acc& acc, int& nin,
                                    unsigned& fl) {
  using Real = RealOf<PREC>;
  Real qq[3], d[3];
  if constexpr (PREC == kNaiveWorld) {
    naive_point(T, e.x, e.y, e.z, qq);
    for (int a = 0; a < 3; ++a) d[a] = (float)e.mean[a] - qq[a];
  } else {
    double q[3];
    transform_exact(T.R, T.t, e.x, e.y, e.z, q);
    for (int a = 0; a < 3; ++a) {
      qq[a] = (Real)q[a];
      d[a] = (Real)(e.mean[a] - q[a]);
    }
  }
  Real o[6];
  const bool ok = fused_inverse<Real>(T.R, e.cov, e.c, o);
  fl |= ok ? 0u : (unsigned)kFlagNonFinite;
  add_point_terms<LIN>(qq, d, o, acc);
  nin += ok ? 1 : 0;
}

// Gradient terms of one inlier (the backward of Eq. (2) with its correspondence held):
// w = R^T Omega d (source frame); the source pose's right-perturbation gradient gains
// 2 w x (mu + C w) (rotation) and -2 w (translation), and the point's gradient is -2 w
// (scaled by the factor's upstream gradient later). Omega is formed in FP64 as everywhere.
struct GradAcc {
  double v[6];
  __device__ void zero() {
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = 0.0;
  }
};

template <int PREC>
__device__ inline void inlier_grad(const RelPose& T, const Inlier& e, GradAcc& acc, int& nin,
                                   unsigned& fl, float* __restrict__ gz) {
  using Real = RealOf<PREC>;
  const float* c = e.c;
  double q[3];
  transform_exact(T.R, T.t, e.x, e.y, e.z, q);
  Real d[3];
  for (int a = 0; a < 3; ++a) d[a] = (Real)(e.mean[a] - q[a]);
  const gptr<float> g = gblw(gz) + 3 * (size_t)(unsigned)e.point;
  Real o[6];
  if (!fused_inverse<Real>(T.R, e.cov, c, o)) {
    fl |= kFlagNonFinite;
    g[0] = 0.0f;
    g[1] = 0.0f;
    g[2] = 0.0f;
    return;
  }
  Real R[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) R[i] = (Real)T.R[i];
  const Real u0 = dot3(o[0], d[0], o[1], d[1], o[2], d[2]);
  const Real u1 = dot3(o[1], d[0], o[3], d[1], o[4], d[2]);
  const Real u2 = dot3(o[2], d[0], o[4], d[1], o[5], d[2]);
  const Real w0 = dot3(R[3], u1, R[0], u0, R[6], u2);
  const Real w1 = dot3(R[4], u1, R[1], u0, R[7], u2);
  const Real w2 = dot3(R[5], u1, R[2], u0, R[8], u2);
  const Real a0 = (Real)e.x + dot3((Real)c[1], w1, (Real)c[0], w0, (Real)c[2], w2);
  const Real a1 = (Real)e.y + dot3((Real)c[3], w1, (Real)c[1], w0, (Real)c[4], w2);
  const Real a2 = (Real)e.z + dot3((Real)c[4], w1, (Real)c[2], w0, (Real)c[5], w2);
  acc.v[0] += 2.0 * (double)det2(w1, a2, w2, a1);
  acc.v[1] += 2.0 * (double)det2(w2, a0, w0, a2);
  acc.v[2] += 2.0 * (double)det2(w0, a1, w1, a0);
  acc.v[3] -= 2.0 * (double)w0;
  acc.v[4] -= 2.0 * (double)w1;
  acc.v[5] -= 2.0 * (double)w2;
  g[0] = (float)(-2.0 * (double)w0);
  g[1] = (float)(-2.0 * (double)w1);
  g[2] = (float)(-2.0 * (double)w2);
  ++nin;
}

// Phase B of one inlier: linearization / evaluation terms, or gradient terms.
template <int PREC, bool LIN, bool GRAD, class Acc>
__device__ inline void phase_b(const RelPose& T, const Inlier& e, Acc& acc, int& nin,
                               unsigned& fl, float* __restrict__ gz) {
  if constexpr (GRAD)
    inlier_grad<PREC>(T, e, acc, nin, fl, gz);
  else
    inlier_terms<PREC, LIN>(T, e, acc, nin, fl);
}

// ------------------------------------------------------------------ one tile

template <int PREC>
struct AccOf {
  using type = AccF32;
};
template <>
struct AccOf<kAccKahan> {
  using type = AccKahan;
};
template <>
struct AccOf<kMathFp64> {
  using type = AccF64;
};

// One wave's part of a tile: chunks of `chunk` points (a multiple of 64 U) every `step` points from
// `base` to `end`, in rows of 64 U points. A row is resolved (phase A) and, whenever at least 64
// inliers are queued, they run with all 64 lanes busy (phase B); the queue tail is flushed at the
// end. The k-th inlier of the wave's sequence goes to lane k mod 64, so a lane's sum depends on
// (base, chunk, step) only, not on U.
template <int PREC, bool LIN, int U, bool DIV, int LAYOUT, bool AOS, bool GRAD, class Acc>
__device__ inline void wave_body(const MapView& m, const RelPose& T,
                                 const float* __restrict__ xyz, const float* __restrict__ cov,
                                 int n, int base, int end, int chunk, int step,
                                 int* __restrict__ corr, Acc& acc, int& nin, unsigned& fl,
                                 const Queue& qe, float* __restrict__ gz) {
  constexpr bool FAST = AOS && PREC != kNaiveWorld;  // only a batch has the error bound
  const int lane = threadIdx.x & 63;
  const Planes P = make_planes(xyz, n);
  int cnt = 0, h = 0;
  Inlier held;  // the last 64 inliers taken from the queue: their terms are formed when the next are
  bool pending = false;
  // positions double-buffered: the next row is loaded while this one is resolved
  Chunk<U> cur;
  cur.load(P, base, lane);
  while (base < end) {
    int next = base + 64 * U;
    h += 64 * U;
    if (h >= chunk) {
      h = 0;
      next += step - chunk;
    }
    Chunk<U> nxt;
    resolve<PREC, DIV, LAYOUT, U, FAST, GRAD>(m, T, cur, nxt, P, next, base, end, lane, qe, cnt,
                                              corr, fl, gz);
    cur = nxt;
    base = next;
    if (cnt >= 64) {
      wave_sync();
      int head = 0;
      for (; cnt - head >= 64; head += 64) {
        Inlier now;
        load_inlier<AOS>(m, cov, n, qe, head + lane, now);
        if (pending) phase_b<PREC, LIN, GRAD>(T, held, acc, nin, fl, gz);
        held = now;
        pending = true;
      }
      const int rem = cnt - head;
      // move the tail to the front (through registers: every lane reads before any writes)
      const int src = min(head + lane, cnt - 1);
      const float ex = qe.e[src].x, ey = qe.e[src].y, ez = qe.e[src].z;
      const int er = qe.e[src].rec, ep = qe.point[src];
      wave_sync();
      if (lane < rem) {
        qe.e[lane].x = ex;
        qe.e[lane].y = ey;
        qe.e[lane].z = ez;
        qe.e[lane].rec = er;
        qe.point[lane] = ep;
      }
      cnt = rem;
      wave_sync();
    }
  }
  wave_sync();
  Inlier last;
  if (lane < cnt) load_inlier<AOS>(m, cov, n, qe, lane, last);
  if (pending) phase_b<PREC, LIN, GRAD>(T, held, acc, nin, fl, gz);
  if (lane < cnt) phase_b<PREC, LIN, GRAD>(T, last, acc, nin, fl, gz);
  wave_sync();
}

// The lane's values in the order of the partial sums (the lane sums' own type: a lane's inlier
// count is exact in either).
template <class Acc>
__device__ inline auto lane_values(const Acc& acc, int nin) {
  using Lane = decltype(acc.get(0));
  struct Values {
    Lane v[32];
  } r;
#pragma unroll
  for (int i = 0; i < kNumAcc; ++i) r.v[i] = acc.get(i);
  r.v[kNumAcc] = (Lane)nin;
#pragma unroll
  for (int i = kPartialStride; i < 32; ++i) r.v[i] = 0;
  return r;
}

// One tile [start, end) of a single factor's source, by one block; writes the tile's partial sums
// (kPartialStride doubles: the 28 sums then the inlier count; evaluate writes only e and the count).
template <int PREC, bool LIN, int BLOCK, int U>
__device__ inline void process_tile(const MapView& m, const RelPose& T,
                                    const float* __restrict__ xyz,
                                    const float* __restrict__ cov, int n, int start, int end,
                                    int* __restrict__ corr, double* __restrict__ partial,
                                    unsigned* flags) {
  __shared__ QueueEntry s_qe[BLOCK / 64][queue_cap<U>()];
  __shared__ int s_qp[BLOCK / 64][queue_cap<U>()];
  const int w = threadIdx.x >> 6;
  typename AccOf<PREC>::type acc;
  acc.zero();
  int nin = 0;
  unsigned fl = 0;
  const Queue qe{s_qe[w], s_qp[w]};
  // uniform: lookup structure and key arithmetic (a multiply when res is a power of 2)
#define VGICP_TILE(DIV, LAYOUT)                                                               \
  wave_body<PREC, LIN, U, DIV, LAYOUT, false, false>(m, T, xyz, cov, n, start + w * 64 * U, end, \
                                                     64 * U, BLOCK * U, corr, acc, nin, fl, qe, \
                                                     nullptr)
  if (m.bricks) {
    if (m.pow2) VGICP_TILE(false, kLayoutGrid); else VGICP_TILE(true, kLayoutGrid);
  } else if (m.slots32) {
    if (m.pow2) VGICP_TILE(false, kLayoutHash32); else VGICP_TILE(true, kLayoutHash32);
  } else {
    if (m.pow2) VGICP_TILE(false, kLayoutHash64); else VGICP_TILE(true, kLayoutHash64);
  }
#undef VGICP_TILE
  if constexpr (LIN) {
    const auto r = lane_values(acc, nin);
    block_sum_store_rs<BLOCK, kPartialStride>(r.v, partial);
  } else {
    double v[2] = {(double)acc.get(kE), (double)nin};
    block_sum_store<BLOCK, 2>(v, partial + kE);
  }
  if (fl) atomicOr(flags, fl);
}

// Adjoint expansion of a factor's 28 target-frame sums (s, in LDS) shared out over the first 64
// threads of the block, an entry per thread: the target-frame blocks H_t, b_t, A = Ad(T_ts),
// G = H_t A; source block A^T G, source gradient -A^T b_t, and for a binary factor the cross
// blocks -G^T, -G and the target block H_t. H is written with row stride ld (12: the batch's
// [F][144] rows, zero blocks for a unary factor; 6 or 12: a single factor's own dimension).
// Every thread of the block must call it (it synchronises).
// Work space of expand_shared in the caller kernel's LDS (kernel-scope arrays: a __shared__
// array inside a device function that several kernels call is laid out once for all of them,
// which sized every such kernel's LDS to the largest).
struct ExpandLds {
  double Ht[36], A[36], G[36], bt[6];
};

__device__ inline void expand_shared(const double* s, const RelPose& T, int binary, double* Hf,
                                     int ld, double* bf, int i, ExpandLds& w) {
  double* Ht = w.Ht;
  double* A = w.A;
  double* G = w.G;
  double* bt = w.bt;
  if (i < 36) {
    const int r = i / 6, c = i % 6;
    const int rr = r % 3, cc = c % 3;
    const int lo = min(rr, cc), hi = max(rr, cc);
    const int sym = lo == 0 ? hi : (lo == 1 ? hi + 2 : 5);
    Ht[i] = r < 3 ? (c < 3 ? s[kHrr + sym] : s[kHrt + 3 * rr + cc])
                  : (c < 3 ? s[kHrt + 3 * cc + rr] : s[kHtt + sym]);
    double a = 0.0;
    if ((r < 3) == (c < 3)) {
      a = T.R[3 * rr + cc];
    } else if (r >= 3) {  // [t]x R: row rr of t x (column cc of R); no local array (an indexed
                          // private array would be moved to LDS, one copy per thread)
      const double c0 = T.R[cc], c1 = T.R[3 + cc], c2 = T.R[6 + cc];
      a = rr == 0 ? T.t[1] * c2 - T.t[2] * c1
                  : (rr == 1 ? T.t[2] * c0 - T.t[0] * c2 : T.t[0] * c1 - T.t[1] * c0);
    }
    A[i] = a;
  }
  if (i < 6) bt[i] = i < 3 ? s[kBr + i] : s[kBt + i - 3];
  __syncthreads();
  if (i < 36) {
    const int r = i / 6, c = i % 6;
    double x = 0.0;
    for (int k = 0; k < 6; ++k) x += Ht[6 * r + k] * A[6 * k + c];
    G[i] = x;
  }
  __syncthreads();
  const int dim = ld == 12 ? 12 : (binary ? 12 : 6);
  for (int e = i; e < dim * dim && i < 64; e += 64) {
    const int R = e / dim, C = e % dim;
    double v = 0.0;
    if (R < 6 && C < 6) {
      for (int k = 0; k < 6; ++k) v += A[6 * k + R] * G[6 * k + C];
    } else if (binary) {
      v = R < 6 ? -G[6 * (C - 6) + R] : (C < 6 ? -G[6 * (R - 6) + C] : Ht[6 * (R - 6) + C - 6]);
    }
    Hf[e] = v;
  }
  if (i < dim) {
    double y = 0.0;
    if (i < 6) {
      for (int k = 0; k < 6; ++k) y += A[6 * k + i] * bt[k];
      y = -y;
    } else if (binary) {
      y = bt[i - 6];
    }
    bf[i] = y;
  }
}

// ------------------------------------------------------------------ single factor

template <int PREC, bool LIN, int BLOCK>
__global__ __launch_bounds__(BLOCK) void plain_tile_kernel(MapView m, RelPose T,
                                                           const float* __restrict__ xyz,
                                                           const float* __restrict__ cov,
                                                           long long n, int tile,
                                                           int* __restrict__ corr,
                                                           double* __restrict__ partials,
                                                           unsigned* flags) {
  const int start = blockIdx.x * tile;
  const int end = (int)min((long long)start + tile, n);
  process_tile<PREC, LIN, BLOCK, 4>(m, T, xyz, cov, (int)n, start, end, corr,
                                    partials + (size_t)blockIdx.x * kPartialStride, flags);
}

// Sums the tile partials (each of the 29 values by 8 threads over every 8th tile, the 8 in
// order: a fixed order) and expands them to H and b (dimension 6 or 12, row stride =
// dimension); writes the cost and inlier count. 256 threads. One block, so a load's latency is what
// it costs: kFinAhead tiles are loaded before they are added (469 tiles: 18.1 us one by
// one, now 6.4).
constexpr int kFinParts = 8, kFinAhead = 16;
template <bool LIN>
__global__ __launch_bounds__(256) void plain_finalize_kernel(const double* __restrict__ partials,
                                                             int ntiles, RelPose T, int binary,
                                                             double* __restrict__ H,
                                                             double* __restrict__ b,
                                                             double* __restrict__ err,
                                                             long long* __restrict__ inliers) {
  __shared__ double part[kPartialStride][kFinParts];
  __shared__ double s[kPartialStride];
  __shared__ ExpandLds ew;
  const int i = threadIdx.x;
  if (i < kPartialStride * kFinParts) {
    const int v = i / kFinParts, q = i % kFinParts;
    double a = 0.0;
    if (LIN || v >= kE)
      for (int t = q; t < ntiles; t += kFinParts * kFinAhead) {
        double p[kFinAhead];
#pragma unroll
        for (int u = 0; u < kFinAhead; ++u)
          p[u] = partials[(long long)min(t + u * kFinParts, ntiles - 1) * kPartialStride + v];
#pragma unroll
        for (int u = 0; u < kFinAhead; ++u)
          if (t + u * kFinParts < ntiles) a += p[u];
      }
    part[v][q] = a;
  }
  __syncthreads();
  if (i < kPartialStride) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < kFinParts; ++q) a += part[i][q];
    s[i] = a;
  }
  __syncthreads();
  if (i == 0) {
    *err = s[kE];
    *inliers = (long long)s[kNumAcc];
  }
  if constexpr (LIN) expand_shared(s, T, binary, H, binary ? 12 : 6, b, i, ew);
}

// ------------------------------------------------------------------ backward

// Per point with a correspondence: w = R^T Omega d; de/domega_s += 2 w x (mu + C w),
// de/drho_s += -2 w, de/dmu = -2 w (times the upstream gradient g).
template <int PREC, int BLOCK>
__global__ __launch_bounds__(BLOCK) void backward_tile_kernel(
    MapView m, RelPose T, const float* __restrict__ xyz, const float* __restrict__ cov,
    long long n, int tile, const int* __restrict__ corr, const double* __restrict__ grad_err,
    double* __restrict__ partials, float* __restrict__ grad_xyz) {
  using Real = RealOf<PREC>;
  const long long start = (long long)blockIdx.x * tile;
  const long long end = min(start + (long long)tile, n);
  const double g = *grad_err;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  const Real* R;
  if constexpr (PREC == kMathFp64)
    R = T.R;
  else
    R = T.Rf;
  for (long long i = start + threadIdx.x; i < end; i += BLOCK) {
    const int v = corr[i];
    if (v < 0 || v >= m.V) {
      if (grad_xyz) {
        grad_xyz[i] = 0.0f;
        grad_xyz[n + i] = 0.0f;
        grad_xyz[2 * n + i] = 0.0f;
      }
      continue;
    }
    const float x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
    float c[6];
    for (int a = 0; a < 6; ++a) c[a] = cov[a * n + i];
    double q[3];
    transform_exact(T.R, T.t, x, y, z, q);
    const VoxelData vd = gbl(m.vox)[v];
    const Real d0 = (Real)(vd.mean[0] - q[0]);
    const Real d1 = (Real)(vd.mean[1] - q[1]);
    const Real d2 = (Real)(vd.mean[2] - q[2]);
    Real o[6];
    if (!fused_inverse<Real>(T.R, vd.cov, c, o)) {
      if (grad_xyz) {
        grad_xyz[i] = 0.0f;
        grad_xyz[n + i] = 0.0f;
        grad_xyz[2 * n + i] = 0.0f;
      }
      continue;
    }
    const Real u0 = dot3(o[1], d1, o[0], d0, o[2], d2);
    const Real u1 = dot3(o[3], d1, o[1], d0, o[4], d2);
    const Real u2 = dot3(o[4], d1, o[2], d0, o[5], d2);
    const Real w0 = dot3(R[3], u1, R[0], u0, R[6], u2);
    const Real w1 = dot3(R[4], u1, R[1], u0, R[7], u2);
    const Real w2 = dot3(R[5], u1, R[2], u0, R[8], u2);
    const Real a0 = (Real)x + dot3((Real)c[1], w1, (Real)c[0], w0, (Real)c[2], w2);
    const Real a1 = (Real)y + dot3((Real)c[3], w1, (Real)c[1], w0, (Real)c[4], w2);
    const Real a2 = (Real)z + dot3((Real)c[4], w1, (Real)c[2], w0, (Real)c[5], w2);
    acc[0] += 2.0 * (double)det2(w1, a2, w2, a1);
    acc[1] += 2.0 * (double)det2(w2, a0, w0, a2);
    acc[2] += 2.0 * (double)det2(w0, a1, w1, a0);
    acc[3] -= 2.0 * (double)w0;
    acc[4] -= 2.0 * (double)w1;
    acc[5] -= 2.0 * (double)w2;
    if (grad_xyz) {
      grad_xyz[i] = (float)(-2.0 * g * (double)w0);
      grad_xyz[n + i] = (float)(-2.0 * g * (double)w1);
      grad_xyz[2 * n + i] = (float)(-2.0 * g * (double)w2);
    }
  }
  block_sum_store<BLOCK, 6>(acc, partials + (long long)blockIdx.x * 6);
}

// g_s = g * sum; binary: g_t = -Ad(T_st)^T g_s with T_st = [R^T | -R^T t].
// Sums the tiles' source gradients, scales by the upstream gradient, forms the target's
// (de/dxi_t = -Ad(T_st)^T de/dxi_s) and maps both to tangent coordinates (J^T g).
__global__ void backward_finalize_kernel(const double* __restrict__ partials, int ntiles,
                                         RelPose T, int binary, TangentMap J,
                                         const double* __restrict__ grad_err,
                                         double* __restrict__ grad_xi) {
  __shared__ double s[12];  // source gradient, then the target's
  const int i = threadIdx.x;
  if (i < 6) {
    double a = 0.0;
    int t = 0;
    for (; t + 16 <= ntiles; t += 16) {  // sixteen loads in flight, added in order
      double v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = partials[(long long)(t + q) * 6 + i];
#pragma unroll
      for (int q = 0; q < 16; ++q) a += v[q];
    }
    for (; t < ntiles; ++t) a += partials[(long long)t * 6 + i];
    s[i] = a * (*grad_err);
  }
  __syncthreads();
  if (binary && i < 6) {
    // column i of A = Ad(T_st), T_st = [R^T | -R^T t]: [[R^T, 0], [[st]x R^T, R^T]]
    double st[3];
    for (int r = 0; r < 3; ++r)
      st[r] = -(T.R[r] * T.t[0] + T.R[3 + r] * T.t[1] + T.R[6 + r] * T.t[2]);
    const int c = i < 3 ? i : i - 3;
    // column c of R^T is row c of R
    const double c0 = c == 0 ? T.R[0] : (c == 1 ? T.R[3] : T.R[6]);
    const double c1 = c == 0 ? T.R[1] : (c == 1 ? T.R[4] : T.R[7]);
    const double c2 = c == 0 ? T.R[2] : (c == 1 ? T.R[5] : T.R[8]);
    const double x0 = st[1] * c2 - st[2] * c1, x1 = st[2] * c0 - st[0] * c2,
                 x2 = st[0] * c1 - st[1] * c0;
    const double g = i < 3 ? (c0 * s[0] + c1 * s[1] + c2 * s[2]) + (x0 * s[3] + x1 * s[4] + x2 * s[5])
                           : c0 * s[3] + c1 * s[4] + c2 * s[5];
    s[6 + i] = -g;
  }
  __syncthreads();
  if (i < (binary ? 12 : 6)) {
    const int h = i < 6 ? 0 : 6, c = i - h;
    const double* Jh = h == 0 ? J.Js : J.Jt;
    double x = s[i];
    if (J.use) {
      x = 0.0;
      for (int r = 0; r < 6; ++r) x += Jh[6 * r + c] * s[h + r];
    }
    grad_xi[i] = x;
  }
}

// ------------------------------------------------------------------ batches

// The FP32 lookup transform and its error bound. With u = 2^-24, A = R / res, s' = t / res - lo and
// M = sum_j |A_j| max|mu_j| + |s'|: rounding A and s' moves s by at most u M, the three FMAs by
// u M (1 + 3 u) each, so s is within 4.01 u M of the real value; the definition's FP64 value is
// within 2^-49 of the magnitudes it sums. 6 u M leaves a third to spare.
// Row r of it; returns the row's bound (NaN where a value is not finite).
__device__ inline double fast_lookup_row(const MapView& m, const float* bx, int r, bool put,
                                         const double* R, double t, RelPose& o) {
  const double lo = (double)m.lo[r];
  const double tk = t * m.inv_res, s = tk - lo;
  double M = fabs(s);
  for (int c = 0; c < 3; ++c) {
    const double A = R[c] * m.inv_res;
    M += fabs(A) * fmax(fabs((double)bx[c]), fabs((double)bx[3 + c]));
    if (put) o.Af[3 * r + c] = (float)A;
  }
  if (put) o.sf[r] = (float)s;
  return 0x1p-24 * 6.0 * M + 0x1p-48 * (M + fabs(tk) + fabs(lo));
}

// Per factor: the relative pose, and whether the source's bounding box (its local frame, the
// eight corners moved by T_ts in FP64 and widened by a margin far above the rounding of any
// point's transform) misses the voxel box of the map: then no point can fall in a voxel and the
// factor's work items are skipped (its sums are zero). Boxes are [lo, hi] per cloud; a cloud
// with a non-finite point has an infinite box and is never skipped, so its error still shows.
// Four lanes a factor, a row of the pose each (the fourth repeats the third's and stores nothing):
// the kernel is one chain of FP64 operations, and the batch waits for it (a lane a factor: 12.5 us for
// 25,440 factors and 4.6 for 24, now 7.4 and 3.5).
constexpr int kPrepBlock = 64;
__global__ __launch_bounds__(kPrepBlock) void batch_prep_kernel(
    const FactorView* __restrict__ F, int nF, const double* __restrict__ poses,
    const float* __restrict__ boxes, int allow_skip, RelPose* __restrict__ rel,
    unsigned long long* __restrict__ heads) {
#pragma clang fp contract(off)
  const int at = blockIdx.x * kPrepBlock + threadIdx.x;
  if (at < kNumXcd) heads[at * kHeadStride] = 0ull;
  const int f = min(at >> 2, nF - 1);  // (lanes past the last factor repeat it)
  const int r = min(at & 3, 2);
  const bool put = (at >> 2) < nF && (at & 3) < 3;
  const double* Tt = poses + 12LL * F[f].target_pose;
  const double* Ts = poses + 12LL * F[f].source_pose;
  const MapView& m = F[f].map;
  RelPose& o = rel[f];
  if (put) rel_pose_row(Tt, Ts, m.inv_res, r, o);
  int skip = 0;
  if (allow_skip && boxes) {
    const float* bx = boxes + 6LL * F[f].source_cloud;
    // the row again: its stores are not read back
    double R[3];
    for (int c = 0; c < 3; ++c) R[c] = (Tt[r] * Ts[c] + Tt[4 + r] * Ts[4 + c]) + Tt[8 + r] * Ts[8 + c];
    const double t = (Tt[r] * (Ts[3] - Tt[3]) + Tt[4 + r] * (Ts[7] - Tt[7])) +
                     Tt[8 + r] * (Ts[11] - Tt[11]);
    double worst = fast_lookup_row(m, bx, r, put, R, t, o);
    double lo = INFINITY, hi = -INFINITY;
    int finite = 1;
    for (int c = 0; c < 8; ++c) {
      const double p[3] = {(double)bx[(c & 1) ? 3 : 0], (double)bx[(c & 2) ? 4 : 1],
                           (double)bx[(c & 4) ? 5 : 2]};
      const double q = ((R[0] * p[0] + R[1] * p[1]) + R[2] * p[2]) + t;
      finite &= isfinite(q) ? 1 : 0;
      lo = fmin(lo, q);
      hi = fmax(hi, q);
    }
    const double mg = 1e-6 * (1.0 + fabs(lo) + fabs(hi));
    const double klo = floor((lo - mg) * m.inv_res), khi = floor((hi + mg) * m.inv_res);
    // the map's voxel coordinates are lo .. lo + ext - 1 (none when the map is empty)
    int miss = khi < (double)m.lo[r] || klo > (double)m.lo[r] + (double)m.ext[r] - 1.0;
    for (int d = 1; d < 4; d <<= 1) {
      const double w = __shfl_xor(worst, d, 64);
      worst = w > worst || !(w >= 0.0) ? w : worst;  // keeps a NaN
      finite &= __shfl_xor(finite, d, 64);
      miss |= __shfl_xor(miss, d, 64);
    }
    skip = finite && miss;
    if (put && r == 0) o.thr = worst < 0.25 ? (float)(0.5 - worst - 0x1p-23) : -1.0f;
  }
  if (put && r == 0) o.skip = skip;
}

void launch_prep(const BatchLaunch& L, int allow_skip, hipStream_t s) {
  batch_prep_kernel<<<(4 * L.F + kPrepBlock - 1) / kPrepBlock, kPrepBlock, 0, s>>>(
      L.factors, L.F, L.poses, L.boxes, allow_skip, L.rel, L.heads);
}

// How a batch's work is cut: `tile` points of a factor per work item, shared by `waves` wave items
// (wave w of a tile takes the chunks of `chunk` points at w * chunk + k * waves * chunk, as the
// waves of one block of the schedule's size would).
struct BatchCut {
  int tile, chunk, waves, wave_shift;
};

// Persistent kernel, a wave item at a time: each wave takes its own items and writes its own
// partial sums, so nothing waits at a barrier (with a block per tile, its reduction, the wait for
// the slowest wave and the next item's dependent loads cost 4.4 us per tile: 0.16 of the global
// batch's time). Block b serves the queue of XCD (b mod 8) first (blocks are dealt to the XCDs
// round-robin, and each queue holds the work of whole groups of factors, so an XCD's L2 sees few
// clouds and maps at a time). The first kStaticShare of a queue is dealt to its waves in turn
// without any atomic; the rest is taken dynamically, by the queue's own waves from the head and
// by helpers from the tail. Same-address atomics are served one every ~15 ns here (20,000 of them
// on one line bounded the batch before), so the counters lie on lines of their own, the next item is
// asked for before the current one is worked on, and a block asks a drained queue once. One
// 64-bit counter per queue holds both ends' counts: an atomic add returns how many items were
// taken before it from either end, so every item is taken exactly once and every wave leaves once
// all queues are drained.
// (Dealing 0.3 of a queue measured best on the global batch, 1,242 us; all dynamic 1,257, 0.5 1,252,
// 0.9 1,466: inliers, and so costs, differ between items.)
constexpr float kStaticShare = 0.3f;

// Waves per SIMD the registers are kept to: 4 (128 registers) where the lane sums are 28 floats, 3
// where they are 56 words.
constexpr int waves_for(int precision) {
  return precision == kAccKahan || precision == kMathFp64 ? 3 : 4;
}

template <int PREC, bool LIN, bool GRAD = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves_for(PREC)))) void
batch_kernel(const FactorView* __restrict__ F, const RelPose* __restrict__ rel,
             const WorkItem* __restrict__ items, const int* __restrict__ seg,
             unsigned long long* __restrict__ heads, BatchCut cut,
             double* __restrict__ partials, unsigned* flags, float* __restrict__ gpts = nullptr) {
  constexpr int U = 2;
  __shared__ QueueEntry s_qe[4][queue_cap<U>()];
  __shared__ int s_qp[4][queue_cap<U>()];
  __shared__ unsigned s_drained;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (threadIdx.x == 0) s_drained = 0u;
  __syncthreads();
  const Queue qe{s_qe[wv], s_qp[wv]};
  const int xcd = blockIdx.x & (kNumXcd - 1);
  const int nw = (int)(gridDim.x / kNumXcd) * 4;           // waves of this queue
  const int rank = (int)(blockIdx.x / kNumXcd) * 4 + wv;
  const int own = (seg[xcd + 1] - seg[xcd]) << cut.wave_shift;
  const int rounds = (int)(kStaticShare * (float)own) / nw;  // items dealt to every wave
  unsigned fl = 0;
  int round = 0, qi = 0;
  bool asked = false;
  unsigned long long old = 0ull;  // lane 0: the counter before this wave's addition
  for (;;) {
    const int x = (xcd + qi) & (kNumXcd - 1);
    const int count = (seg[x + 1] - seg[x]) << cut.wave_shift;
    // the part of queue x that its own waves do not take in turn starts here
    const int first = ((int)(kStaticShare * (float)count) / nw) * nw;
    const unsigned long long inc = qi == 0 ? 1ull : (1ull << 32);
    int idx;
    if (round < rounds) {
      idx = round * nw + rank;
      ++round;
    } else {
      if (!asked) {
        if (__builtin_amdgcn_readfirstlane((int)((s_drained >> x) & 1u))) {
          if (++qi == kNumXcd) break;
          continue;
        }
        if (lane == 0) old = atomicAdd(&heads[x * kHeadStride], inc);
      }
      asked = false;
      const int from_head = __builtin_amdgcn_readfirstlane((int)(unsigned)old);
      const int from_tail = __builtin_amdgcn_readfirstlane((int)(unsigned)(old >> 32));
      if ((long long)from_head + from_tail >= (long long)(count - first)) {
        if (lane == 0) atomicOr(&s_drained, 1u << x);
        if (++qi == kNumXcd) break;
        continue;
      }
      idx = qi == 0 ? first + from_head : count - 1 - from_tail;
    }
    if (round >= rounds) {  // ask for the next item now
      if (lane == 0) old = atomicAdd(&heads[x * kHeadStride], inc);
      asked = true;
    }
    const int it = seg[x] + (idx >> cut.wave_shift), w = idx & (cut.waves - 1);
    const int wf = __builtin_amdgcn_readfirstlane(items[it].factor);
    const int wt = __builtin_amdgcn_readfirstlane(items[it].tile);
    const RelPose& T = rel[wf];
    if (__builtin_amdgcn_readfirstlane(T.skip)) continue;  // the finalize writes zeros
    const FactorView& f = F[wf];
    const MapView& m = f.map;
    const int start = wt * cut.tile;
    const int end = (int)min((long long)start + cut.tile, f.n);
    double* partial = partials + ((size_t)(f.tile_base + wt) * cut.waves + w) * kPartialStride;
    typename std::conditional<GRAD, GradAcc, typename AccOf<PREC>::type>::type acc;
    acc.zero();
    int nin = 0;
    float* gz = GRAD ? gpts + 3 * (size_t)f.gbase : nullptr;
#define VGICP_WAVE(LAYOUT)                                                                      \
  wave_body<PREC, LIN, U, false, LAYOUT, true, GRAD>(m, T, f.xyz, f.cov6, (int)f.n,               \
                                                   start + w * cut.chunk, end, cut.chunk,       \
                                                   cut.waves * cut.chunk, nullptr, acc, nin, fl, \
                                                   qe, gz)
    if (m.bricks)
      VGICP_WAVE(kLayoutGrid);
    else if (m.slots32)
      VGICP_WAVE(kLayoutHash32);
    else
      VGICP_WAVE(kLayoutHash64);
#undef VGICP_WAVE
    if constexpr (GRAD) {
      double v[7];
#pragma unroll
      for (int i = 0; i < 6; ++i) v[i] = acc.v[i];
      v[6] = (double)nin;
      wave_sum_store<7>(v, partial);
    } else if constexpr (LIN) {
      const auto r = lane_values(acc, nin);
      const double v = wave_sum_rs(r.v);
      if ((lane & 1) == 0 && (lane >> 1) < kPartialStride) partial[lane >> 1] = v;
    } else {
      double v[2] = {(double)acc.get(kE), (double)nin};
      wave_sum_store<2>(v, partial + kE);
    }
  }
  if (fl) atomicOr(flags, fl);
}

// Points [lo, end) of a source that have a voxel in the map (a loop per lookup structure: one loop
// around all three holds the scalars of each).
template <int LAYOUT>
__device__ inline int count_points(const MapView& m, const RelPose& T, const Planes& P, int lo,
                                   int end, int lane, unsigned& fl) {
  constexpr int U = 2;
  const Queue none{nullptr, nullptr};
  int cnt = 0;
  Chunk<U> cur, nxt;
  cur.load(P, lo, lane);
  for (int base = lo; base < end; base += 64 * U) {
    resolve<kCountOnly, false, LAYOUT, U, true>(m, T, cur, nxt, P, base + 64 * U, base, end, lane,
                                                none, cnt, nullptr, fl);
    cur = nxt;
  }
  return cnt;
}

// Overlap counts: every point's voxel, nothing else. The counts are whole numbers, so the cut is
// free: a wave takes a tile's share of 1 / waves in one piece, the items are dealt to the waves in
// turn (their cost is even: no counter is shared), 64 items' skip flags are read at once, and the
// few registers leave 8 waves per SIMD.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void batch_count_kernel(
    const FactorView* __restrict__ F, const RelPose* __restrict__ rel,
    const WorkItem* __restrict__ items, const int* __restrict__ seg, BatchCut cut,
    int* __restrict__ counts, unsigned* flags) {
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int xcd = blockIdx.x & (kNumXcd - 1);
  const int nw = (int)(gridDim.x / kNumXcd) * 4;
  const int rank = (int)(blockIdx.x / kNumXcd) * 4 + wv;
  const int first = seg[xcd], own = (seg[xcd + 1] - first) << cut.wave_shift;
  const int share = cut.tile >> cut.wave_shift;
  unsigned fl = 0;
  for (int at = rank; at < own; at += 64 * nw) {
    // lane l looks at item at + l * nw
    const long long mine = (long long)at + (long long)lane * nw;
    const bool live = mine < own && rel[items[first + (int)(mine >> cut.wave_shift)].factor].skip == 0;
    for (unsigned long long todo = __ballot(live); todo != 0ull; todo &= todo - 1ull) {
      const int idx = at + __builtin_ctzll(todo) * nw;
      const int it = first + (idx >> cut.wave_shift), w = idx & (cut.waves - 1);
      const int wf = __builtin_amdgcn_readfirstlane(items[it].factor);
      const int wt = __builtin_amdgcn_readfirstlane(items[it].tile);
      const RelPose& T = rel[wf];
      const FactorView& f = F[wf];
      const MapView& m = f.map;
      const Planes P = make_planes(f.xyz, (int)f.n);
      const int lo = wt * cut.tile + w * share;
      const int end = (int)min((long long)lo + share, f.n);
      const int cnt = m.bricks    ? count_points<kLayoutGrid>(m, T, P, lo, end, lane, fl)
                      : m.slots32 ? count_points<kLayoutHash32>(m, T, P, lo, end, lane, fl)
                                  : count_points<kLayoutHash64>(m, T, P, lo, end, lane, fl);
      if (lane == 0) counts[(size_t)(f.tile_base + wt) * cut.waves + w] = cnt;
    }
  }
  if (fl) atomicOr(flags, fl);
}

// Inliers and overlap rate of every factor: one wave adds a factor's counts.
__global__ __launch_bounds__(256) void batch_count_finalize_kernel(
    const FactorView* __restrict__ F, const RelPose* __restrict__ rel, int nF, int waves,
    const int* __restrict__ counts, double* __restrict__ rates, long long* __restrict__ inliers) {
  const int f = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (f >= nF) return;
  const int n = rel[f].skip ? 0 : F[f].ntiles * waves;
  const int* c = counts + (size_t)F[f].tile_base * waves;
  int a = 0;  // at most 2^30 points
  for (int i = lane; i < n; i += 64) a += c[i];
  for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
  if (lane == 0) {
    rates[f] = F[f].n > 0 ? (double)a / (double)F[f].n : 0.0;
    inliers[f] = a;
  }
}

// A factor's tiles in order, each the sum of its waves in order.
__device__ inline double sum_tiles(const double* __restrict__ partials, long long base, int nt,
                                   int waves, int i) {
  const double* p = partials + base * waves * kPartialStride + i;
  double a = 0.0;
  auto add = [&](auto waves_tag) {
    constexpr int W = decltype(waves_tag)::value, kAhead = 16 / W;  // sixteen loads in flight
    for (int t = 0; t < nt; t += kAhead) {
      double v[kAhead][W];
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
#pragma unroll
        for (int w = 0; w < W; ++w)
          v[u][w] = p[((long long)min(t + u, nt - 1) * W + w) * kPartialStride];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        double s = v[u][0];
#pragma unroll
        for (int w = 1; w < W; ++w) s += v[u][w];
        if (t + u < nt) a += s;
      }
    }
  };
  if (waves == 8)
    add(std::integral_constant<int, 8>{});
  else
    add(std::integral_constant<int, 4>{});
  return a;
}

template <bool LIN>
__global__ __launch_bounds__(64) void batch_finalize_kernel(const FactorView* __restrict__ F,
                                      const RelPose* __restrict__ rel,
                                      const double* __restrict__ partials, int waves,
                                      double* __restrict__ H, double* __restrict__ b,
                                      double* __restrict__ err, long long* __restrict__ inliers) {
  __shared__ double s[kPartialStride];
  __shared__ ExpandLds ew;
  const int f = blockIdx.x;
  const int i = threadIdx.x;
  const int base = F[f].tile_base, nt = rel[f].skip ? 0 : F[f].ntiles;
  if (i < kPartialStride && (LIN || i >= kE)) s[i] = sum_tiles(partials, base, nt, waves, i);
  __syncthreads();
  if (i == 0) {
    err[f] = s[kE];
    inliers[f] = (long long)s[kNumAcc];
  }
  if constexpr (LIN) expand_shared(s, rel[f], F[f].binary, H + 144LL * f, 12, b + 12LL * f, i, ew);
}

// ------------------------------------------------------------------ batched backward

// Per factor: the source pose's gradient summed over the tiles in order, scaled by the
// factor's upstream gradient; a binary factor's target gradient is -Ad(T_st)^T of it.
// gf[f] = [source | target] (the target half is zero for a unary factor).
__global__ void batch_grad_finalize_kernel(const FactorView* __restrict__ F,
                                           const RelPose* __restrict__ rel,
                                           const double* __restrict__ partials, int waves,
                                           const double* __restrict__ grad_err,
                                           double* __restrict__ gf) {
  __shared__ double s[6];
  const int f = blockIdx.x;
  const int i = threadIdx.x;
  const int base = F[f].tile_base, nt = rel[f].skip ? 0 : F[f].ntiles;
  if (i < 6) s[i] = sum_tiles(partials, base, nt, waves, i) * grad_err[f];
  __syncthreads();
  if (i < 12) {
    double v = 0.0;
    if (i < 6) {
      v = s[i];
    } else if (F[f].binary) {
      // column c of A = Ad(T_st) = [R' 0; [t']x R' R'], T_st = T_ts^-1 = [R' = R^T | t' = -R^T t]
      // (formed by its lane: an indexed 6 x 6 array would lie in scratch memory)
      const RelPose& T = rel[f];
      const int c = (i - 6) % 3;
      const double c0 = T.R[3 * c], c1 = T.R[3 * c + 1], c2 = T.R[3 * c + 2];
      double st[3];
      for (int r = 0; r < 3; ++r)
        st[r] = -(T.R[r] * T.t[0] + T.R[3 + r] * T.t[1] + T.R[6 + r] * T.t[2]);
      if (i < 9) {
        v = c0 * s[0] + c1 * s[1] + c2 * s[2];
        v += (st[1] * c2 - st[2] * c1) * s[3];
        v += (st[2] * c0 - st[0] * c2) * s[4];
        v += (st[0] * c1 - st[1] * c0) * s[5];
      } else {
        v = c0 * s[3] + c1 * s[4] + c2 * s[5];
      }
      v = -v;
    }
    gf[12LL * f + i] = v;
  }
}

// Per pose and tangent entry: the factors' gradients summed in factor order (deterministic).
__global__ void batch_grad_pose_kernel(const int* __restrict__ bptr,
                                       const int* __restrict__ bcontrib,
                                       const double* __restrict__ gf, int P,
                                       double* __restrict__ grad_poses) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 6 * P) return;
  const int p = t / 6, r = t % 6;
  double s = 0.0;
#pragma unroll 8
  for (int q = bptr[p]; q < bptr[p + 1]; ++q) {
    const int w = bcontrib[q];
    s += gf[12LL * (w >> 1) + 6 * (w & 1) + r];
  }
  grad_poses[t] = s;
}

// Per source cloud (blockIdx.y) and point of its spatial order: the gradients of the factors
// that read it, summed in factor order and scaled by their upstream gradients, written to the
// caller's [3][n] array at the point's original index. A skipped factor has no inlier. A lane waits
// for memory only, so the values of kGradAhead factors are loaded before they are added
// (256 factors, 18,000 points a cloud: 20.8 us to 18.3, near the rate of memory).
constexpr int kGradAhead = 8;
__global__ __launch_bounds__(256) void batch_grad_points_kernel(
    const FactorView* __restrict__ F, const RelPose* __restrict__ rel,
    const int* __restrict__ cptr, const int* __restrict__ cfac,
    const long long* __restrict__ cloud_n, const long long* __restrict__ cloud_off,
    const int* __restrict__ perm, float* const* __restrict__ out,
    const double* __restrict__ grad_err, const float* __restrict__ gpts) {
  const int c = blockIdx.y;
  const long long n = cloud_n[c];
  float* o = out[c];
  if (!o) return;
  const int j0 = cptr[c], j1 = cptr[c + 1];
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (long long)gridDim.x * blockDim.x) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int j = j0; j < j1; j += kGradAhead) {
      // no branch around the loads: past the last factor the last one's are loaded again, a skipped
      // factor's rows hold old values, and neither is added
      int f[kGradAhead];
      double g[kGradAhead];
      float v[kGradAhead][3];
#pragma unroll
      for (int u = 0; u < kGradAhead; ++u) f[u] = cfac[min(j + u, j1 - 1)];
#pragma unroll
      for (int u = 0; u < kGradAhead; ++u) {
        const gptr<const float> p = gbl(gpts) + 3 * (size_t)(F[f[u]].gbase + k);
        v[u][0] = p[0];
        v[u][1] = p[1];
        v[u][2] = p[2];
      }
#pragma unroll
      for (int u = 0; u < kGradAhead; ++u) {
        const bool add = j + u < j1 && rel[f[u]].skip == 0;
        g[u] = add ? grad_err[f[u]] : 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) v[u][a] = add ? v[u][a] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < kGradAhead; ++u) {
        s0 += g[u] * (double)v[u][0];
        s1 += g[u] * (double)v[u][1];
        s2 += g[u] * (double)v[u][2];
      }
    }
    // a cloud no factor reads was never put in spatial order: its points keep their index
    const long long i = j0 == j1 ? k : perm[cloud_off[c] + k];
    o[i] = (float)s0;
    o[n + i] = (float)s1;
    o[2 * n + i] = (float)s2;
  }
}

// ------------------------------------------------------------------ dispatch

template <int PREC, bool LIN>
void launch_plain_t(const MapView& m, const RelPose& T, const float* xyz, const float* cov,
                    int64_t n, int binary, double* partials, int ntiles, int tile,
                    int32_t* corr, unsigned* flags, double* H, double* b, double* err,
                    int64_t* inliers, hipStream_t s) {
  if (ntiles > 0)
    plain_tile_kernel<PREC, LIN, 256><<<ntiles, 256, 0, s>>>(m, T, xyz, cov, n, tile, corr,
                                                             partials, flags);
  plain_finalize_kernel<LIN><<<1, 256, 0, s>>>(partials, ntiles, T, binary, H, b, err,
                                             reinterpret_cast<long long*>(inliers));
}

BatchCut cut_of(const BatchLaunch& L) {
  return {L.tile, 64 * L.lookahead, L.block / 64, L.block == 512 ? 3 : 2};
}

template <int PREC>
int resident(const BatchLaunch& L) {
  return batch_grid(L.grid, L.total_tiles, L.block, L.cus, PREC);
}

template <int PREC, bool LIN>
void launch_batch_t(const BatchLaunch& L, hipStream_t s) {
  const BatchCut cut = cut_of(L);
  launch_prep(L, PREC != kNaiveWorld, s);
  batch_kernel<PREC, LIN><<<resident<PREC>(L), 256, 0, s>>>(L.factors, L.rel, L.items, L.seg, L.heads, cut,
                                                 L.partials, L.flags);
  batch_finalize_kernel<LIN><<<L.F, 64, 0, s>>>(L.factors, L.rel, L.partials, cut.waves, L.H, L.b,
                                                L.err, reinterpret_cast<long long*>(L.inliers));
}

void launch_batch_count(const BatchLaunch& L, hipStream_t s) {
  const BatchCut cut = cut_of(L);  // 8 blocks of 4 waves fill a CU's 32 wave slots
  int* counts = reinterpret_cast<int*>(L.partials);
  launch_prep(L, 1, s);
  batch_count_kernel<<<8 * L.cus / kNumXcd * kNumXcd, 256, 0, s>>>(L.factors, L.rel, L.items, L.seg, cut, counts,
                                                  L.flags);
  batch_count_finalize_kernel<<<(L.F + 3) / 4, 256, 0, s>>>(
      L.factors, L.rel, L.F, cut.waves, counts, L.err, reinterpret_cast<long long*>(L.inliers));
}

}  // namespace

// The schedule's grid, but no more blocks than fit the chip together: a wave of a later round would
// start on its dealt items when everyone else is done (global batch, 6 blocks per CU instead of 4:
// 1,371 us instead of 1,242).
int batch_grid(int grid, int total_tiles, int block, int cus, int precision) {
  const int need = (total_tiles * (block / 64) + 3) / 4;  // a wave item per wave at least
  const int most = std::min(grid, cus * waves_for(precision));
  return std::max((std::min(need, most) + kNumXcd - 1) / kNumXcd, 1) * kNumXcd;
}

void launch_plain(const MapView& m, const RelPose& T, const float* xyz, const float* cov,
                  int64_t n, int binary, int precision, bool linearize, double* partials,
                  int ntiles, int tile, int32_t* corr, unsigned* flags, double* H, double* b,
                  double* err, int64_t* inliers, hipStream_t s) {
#define VGICP_PLAIN(P)                                                                        \
  (linearize ? launch_plain_t<P, true>(m, T, xyz, cov, n, binary, partials, ntiles, tile, corr, \
                                       flags, H, b, err, inliers, s)                          \
             : launch_plain_t<P, false>(m, T, xyz, cov, n, binary, partials, ntiles, tile,    \
                                        corr, flags, H, b, err, inliers, s))
  switch (precision) {
    case kAccKahan: VGICP_PLAIN(kAccKahan); break;
    case kNaiveWorld: VGICP_PLAIN(kNaiveWorld); break;
    case kMathFp64: VGICP_PLAIN(kMathFp64); break;
    default: VGICP_PLAIN(kAccFp64); break;
  }
#undef VGICP_PLAIN
}

void launch_backward(const MapView& m, const RelPose& T, const TangentMap& J, const float* xyz,
                     const float* cov, int64_t n, int binary, int precision,
                     const int32_t* corr, const double* grad_err, double* partials, int ntiles,
                     int tile, double* grad_xi, float* grad_xyz, hipStream_t s) {
  if (ntiles > 0) {
    if (precision == kMathFp64)
      backward_tile_kernel<kMathFp64, 256><<<ntiles, 256, 0, s>>>(
          m, T, xyz, cov, n, tile, corr, grad_err, partials, grad_xyz);
    else
      backward_tile_kernel<kAccFp64, 256><<<ntiles, 256, 0, s>>>(
          m, T, xyz, cov, n, tile, corr, grad_err, partials, grad_xyz);
  }
  backward_finalize_kernel<<<1, 64, 0, s>>>(partials, ntiles, T, binary, J, grad_err, grad_xi);
}

namespace {
template <int PREC>
void launch_batch_grad_t(const BatchLaunch& L, const BatchGrad& G, hipStream_t s) {
  const BatchCut cut = cut_of(L);
  launch_prep(L, 1, s);
  batch_kernel<PREC, false, true><<<resident<PREC>(L), 256, 0, s>>>(L.factors, L.rel, L.items, L.seg,
                                                         L.heads, cut, L.partials, L.flags, G.gpts);
  batch_grad_finalize_kernel<<<L.F, 64, 0, s>>>(L.factors, L.rel, L.partials, cut.waves,
                                                G.grad_err, G.gf);
  if (G.P > 0)
    batch_grad_pose_kernel<<<(6 * G.P + 255) / 256, 256, 0, s>>>(G.bptr, G.bcontrib, G.gf, G.P,
                                                               G.grad_poses);
  if (G.n_clouds > 0 && G.max_n > 0) {
    const long long gx = std::min<long long>((G.max_n + 255) / 256, 4096);
    batch_grad_points_kernel<<<dim3((unsigned)gx, (unsigned)G.n_clouds), 256, 0, s>>>(
        L.factors, L.rel, G.cptr, G.cfac, G.cloud_n, G.cloud_off, G.perm, G.out, G.grad_err,
        G.gpts);
  }
}

}  // namespace

void launch_batched_backward(const BatchLaunch& L, const BatchGrad& G, hipStream_t s) {
  if (L.precision == kMathFp64)
    launch_batch_grad_t<kMathFp64>(L, G, s);
  else
    launch_batch_grad_t<kAccFp64>(L, G, s);
}

void launch_batched(const BatchLaunch& L, hipStream_t s) {
#define VGICP_BATCH(P) \
  (L.linearize ? launch_batch_t<P, true>(L, s) : launch_batch_t<P, false>(L, s))
  switch (L.precision) {
    case kAccKahan: VGICP_BATCH(kAccKahan); break;
    case kNaiveWorld: VGICP_BATCH(kNaiveWorld); break;
    case kMathFp64: VGICP_BATCH(kMathFp64); break;
    case kCountOnly: launch_batch_count(L, s); break;
    default: VGICP_BATCH(kAccFp64); break;
  }
#undef VGICP_BATCH
}

}  // namespace vgicp
