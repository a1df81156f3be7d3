// IMU preintegration factor of Sec. III-B (Eqs. (4)-(9)), batched over factors, FP64.
//   * preintegration: per factor, its samples in order (Eqs. (4)-(6) from the body frame at
//     time i, no gravity): dR <- dR Exp((w - b_w) dt), dv <- dv + dR (a - b_a) dt,
//     dp <- dp + dv dt + dR (a - b_a) dt^2 / 2, with the covariance of the preintegration noise
//     (dphi, dv, dp) propagated to first order, S <- A S A^T + B Q B^T (the on-manifold
//     preintegration the section cites);
//   * linearization: residual r = [Log(dR^T R_i^T R_j); R_i^T (v_j - v_i - g dt) - dv;
//     R_i^T (t_j - t_i - v_i dt - g dt^2 / 2) - dp] (Eqs. (7)-(9)), its Jacobian over
//     [xi_i, v_i, xi_j, v_j] (right perturbation of the poses, additive velocities), whitened by
//     the Cholesky factor of S: H = J^T S^-1 J, b = J^T S^-1 r, e = r^T S^-1 r.
//   * with bias states: the preintegration's derivatives with respect to the biases, the
//     first-order bias correction and the bias random walk (15 residuals, 30 unknowns).
// A factor holds tens to hundreds of samples and a graph a few thousand factors: 16 lanes per factor
// for the preintegration, one thread, everything in registers, for the 18-unknown factor, eight
// factors per block for the 30-unknown one (their 900-entry Hessians are formed in parallel).
#include <cmath>

#include "internal.h"

namespace vgicp {
namespace {

constexpr int kImuBlock = 64;

__device__ inline void hat3(const double w[3], double K[3][3]) {
  K[0][0] = 0.0;
  K[0][1] = -w[2];
  K[0][2] = w[1];
  K[1][0] = w[2];
  K[1][1] = 0.0;
  K[1][2] = -w[0];
  K[2][0] = -w[1];
  K[2][1] = w[0];
  K[2][2] = 0.0;
}

// Exp(w) (Rodrigues), and with J non-null the right Jacobian J_r(w) (series near zero).
__device__ inline void so3_exp_jr(const double w[3], double E[3][3], double (*J)[3]) {
  const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
  const double th = sqrt(th2);
  double K[3][3], K2[3][3];
  hat3(w, K);
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) K2[r][c] = K[r][0] * K[0][c] + K[r][1] * K[1][c] + K[r][2] * K[2][c];
  double a, b, ja, jb;  // E = I + a K + b K^2, J_r = I - ja K + jb K^2
  if (th < 1e-8) {
    a = 1.0;
    b = 0.5;
    ja = 0.5;
    jb = 1.0 / 6.0;
  } else {
    const double s = sin(th), c = cos(th);
    a = s / th;
    b = (1.0 - c) / th2;
    ja = b;
    jb = (th - s) / (th2 * th);
  }
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double id = r == c ? 1.0 : 0.0;
      E[r][c] = id + a * K[r][c] + b * K2[r][c];
      if (J) J[r][c] = id - ja * K[r][c] + jb * K2[r][c];
    }
}

// Log(R) as a rotation vector (angle below pi), and J_r^-1 of that vector.
__device__ inline void so3_log_jrinv(const double R[3][3], double w[3], double Ji[3][3]) {
  const double c = fmin(fmax((R[0][0] + R[1][1] + R[2][2] - 1.0) * 0.5, -1.0), 1.0);
  const double th = acos(c);
  const double v[3] = {R[2][1] - R[1][2], R[0][2] - R[2][0], R[1][0] - R[0][1]};
  const double f = th < 1e-8 ? 0.5 : th / (2.0 * sin(th));
#pragma unroll
  for (int i = 0; i < 3; ++i) w[i] = f * v[i];
  double K[3][3], K2[3][3];
  hat3(w, K);
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc)
      K2[r][cc] = K[r][0] * K[0][cc] + K[r][1] * K[1][cc] + K[r][2] * K[2][cc];
  const double g = th < 1e-8 ? 1.0 / 12.0
                             : 1.0 / (th * th) - (1.0 + cos(th)) / (2.0 * th * sin(th));
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) Ji[r][cc] = (r == cc ? 1.0 : 0.0) + 0.5 * K[r][cc] + g * K2[r][cc];
}

// Broadcast of lane N of every row of 16 lanes (a register move).
template <int N>
__device__ inline double row_lane(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + N, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + N, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Preintegration, 16 lanes per factor: the mean and the sample's matrices are the same in all of
// them; lane c < 9 carries column c of the noise covariance S, lanes 9 .. 14 the columns of the
// mean's derivatives J with respect to the biases (b_a, b_w). With A the error propagation of a
// sample (rows (E^T, 0, 0), (M1, I, 0), (M1 dt / 2, I dt, I), M1 = -dR [a]x dt) both go through the
// same product, A S and A J; then S <- (A S) A^T + B Q B^T (columns 0 .. 2 of A S broadcast along
// the row) and J gains -J_r dt (rotation, b_w), -dR dt and -dR dt^2 / 2 (velocity and position, b_a).
// What depends on one sample only (its exponential, right Jacobian and noise) is computed for 16
// samples at once, one per lane, and read back from LDS: done in turn by all lanes it was most of a
// sample's 3.6 us. A thread per factor was 63 waves of 1,700 FP64 instructions a sample on a
// quarter of the CUs and a second launch for the derivatives: 4,000 factors of 20 samples took 52 + 25 us.
constexpr int kImuLanes = 16;
__global__ __launch_bounds__(kImuBlock) void imu_preintegrate_kernel(
    const double* __restrict__ imu, long long m, const long long* __restrict__ seg, int F,
    const double* __restrict__ bias, double sg2, double sa2, double* __restrict__ pre,
    double* __restrict__ cov, double* __restrict__ jac, unsigned* __restrict__ flags) {
  __shared__ double sS[kImuBlock / kImuLanes][9][9];
  __shared__ double sM[kImuBlock / kImuLanes][kImuLanes][24];  // E, J_r, a, dt, gyro and acc noise
  const int f = (int)(((long long)blockIdx.x * kImuBlock + threadIdx.x) / kImuLanes);
  const int c = threadIdx.x & (kImuLanes - 1), slot = threadIdx.x / kImuLanes;
  if (f >= F) return;  // whole rows
  const long long k0 = seg[f], k1 = seg[f + 1];
  if (k0 < 0 || k1 < k0 || k1 > m) {
    if (c == 0) atomicOr(flags, kFlagBadIndex);
    return;
  }
  const double ba[3] = {bias[6 * f], bias[6 * f + 1], bias[6 * f + 2]};
  const double bw[3] = {bias[6 * f + 3], bias[6 * f + 4], bias[6 * f + 5]};
  double dR[3][3] = {{1.0, 0.0, 0.0}, {0.0, 1.0, 0.0}, {0.0, 0.0, 1.0}};
  double dv[3] = {0.0, 0.0, 0.0}, dp[3] = {0.0, 0.0, 0.0}, T = 0.0;
  double x[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // this lane's column
  // the column's place in its 3 x 3 block, and which block: S 0 .. 2, J 3 (b_a), 4 (b_w), 5 none
  const int cc = c % 3, blk = c / 3;
  bool bad = false;
  for (long long k = k0; k < k1; ++k) {
    const int at_lane = (int)((k - k0) & (kImuLanes - 1));
    if (at_lane == 0) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (k + c < k1) {
        const double* row = imu + 7 * (k + c);
        const double dt = row[6];
        if (!(dt > 0.0) || !isfinite(dt)) bad = true;
        const double wt[3] = {(row[0] - bw[0]) * dt, (row[1] - bw[1]) * dt, (row[2] - bw[2]) * dt};
        double E[3][3], Jr[3][3];
        so3_exp_jr(wt, E, Jr);
        double* o = sM[slot][c];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            o[3 * r + q] = E[r][q];
            o[9 + 3 * r + q] = Jr[r][q];
          }
#pragma unroll
        for (int r = 0; r < 3; ++r) o[18 + r] = row[3 + r] - ba[r];
        o[21] = dt;
        o[22] = sg2 / dt * dt * dt;
        o[23] = sa2 / dt * dt * dt;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    const double* o = sM[slot][at_lane];
    double E[3][3], Jr[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        E[r][q] = o[3 * r + q];
        Jr[r][q] = o[9 + 3 * r + q];
      }
    const double at[3] = {o[18], o[19], o[20]};
    const double dt = o[21], qg = o[22], qa = o[23];
    // M1 = -dR [a]x dt
    double Ka[3][3], M1[3][3];
    hat3(at, Ka);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        M1[r][q] = -(dR[r][0] * Ka[0][q] + dR[r][1] * Ka[1][q] + dR[r][2] * Ka[2][q]) * dt;
    // column of A S or A J
    double y[9];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const double mm = M1[r][0] * x[0] + M1[r][1] * x[1] + M1[r][2] * x[2];
      y[r] = E[0][r] * x[0] + E[1][r] * x[1] + E[2][r] * x[2];
      y[3 + r] = mm + x[3 + r];
      y[6 + r] = 0.5 * dt * mm + dt * x[3 + r] + x[6 + r];
    }
    // this column's coefficients on columns 0 .. 2 of A S: row c of A's first block column, and its
    // column of dR and J_r
    double a0[3], dRc[3], Jrc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double e = cc == 0 ? E[q][0] : (cc == 1 ? E[q][1] : E[q][2]);
      const double mq = cc == 0 ? M1[0][q] : (cc == 1 ? M1[1][q] : M1[2][q]);
      a0[q] = blk == 0 ? e : (blk == 1 ? mq : 0.5 * dt * mq);
      dRc[q] = cc == 0 ? dR[q][0] : (cc == 1 ? dR[q][1] : dR[q][2]);
      Jrc[q] = cc == 0 ? Jr[q][0] : (cc == 1 ? Jr[q][1] : Jr[q][2]);
    }
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      // (A S) A^T: the position columns also take dt times the velocity column three lanes below
      const double z = a0[0] * row_lane<0>(y[r]) + a0[1] * row_lane<1>(y[r]) + a0[2] * row_lane<2>(y[r]);
      const double vel = __shfl_up(y[r], 3, kImuLanes);
      x[r] = blk == 0 ? z : (blk == 1 ? z + y[r] : (blk == 2 ? z + dt * vel + y[r] : y[r]));
    }
    // + B Q B^T (gyro noise through J_r dt, accelerometer noise through dR dt and dR dt^2 / 2), or the
    // derivatives' own terms
    double jj[3], rr[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      // column cc of J_r J_r^T and dR dR^T: row r times row cc
      const double j0 = cc == 0 ? Jr[0][0] : (cc == 1 ? Jr[1][0] : Jr[2][0]);
      const double j1 = cc == 0 ? Jr[0][1] : (cc == 1 ? Jr[1][1] : Jr[2][1]);
      const double j2 = cc == 0 ? Jr[0][2] : (cc == 1 ? Jr[1][2] : Jr[2][2]);
      const double r0 = cc == 0 ? dR[0][0] : (cc == 1 ? dR[1][0] : dR[2][0]);
      const double r1 = cc == 0 ? dR[0][1] : (cc == 1 ? dR[1][1] : dR[2][1]);
      const double r2 = cc == 0 ? dR[0][2] : (cc == 1 ? dR[1][2] : dR[2][2]);
      jj[r] = Jr[r][0] * j0 + Jr[r][1] * j1 + Jr[r][2] * j2;
      rr[r] = dR[r][0] * r0 + dR[r][1] * r1 + dR[r][2] * r2;
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const double rot = blk == 0 ? qg * jj[r] : (blk == 4 ? -Jrc[r] * dt : 0.0);
      const double vel = blk == 1 ? qa * rr[r]
                                  : (blk == 2 ? 0.5 * dt * qa * rr[r] : (blk == 3 ? -dRc[r] * dt : 0.0));
      const double pos = blk == 1 ? 0.5 * dt * qa * rr[r]
                                  : (blk == 2 ? 0.25 * dt * dt * qa * rr[r]
                                              : (blk == 3 ? -0.5 * dRc[r] * dt * dt : 0.0));
      x[r] += rot;
      x[3 + r] += vel;
      x[6 + r] += pos;
    }
    // the mean
    double ra[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) ra[r] = dR[r][0] * at[0] + dR[r][1] * at[1] + dR[r][2] * at[2];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      dp[r] += dv[r] * dt + 0.5 * ra[r] * dt * dt;
      dv[r] += ra[r] * dt;
    }
    double nR[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        nR[r][q] = dR[r][0] * E[0][q] + dR[r][1] * E[1][q] + dR[r][2] * E[2][q];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int q = 0; q < 3; ++q) dR[r][q] = nR[r][q];
    T += dt;
  }
  if (bad) atomicOr(flags, kFlagNonFinite);
  if (c == 15) {
    double* o = pre + 16 * (long long)f;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
      for (int q = 0; q < 3; ++q) o[3 * r + q] = dR[r][q];
      o[9 + r] = dv[r];
      o[12 + r] = dp[r];
    }
    o[15] = T;
  }
  if (jac && c >= 9 && c < 15) {
    double* o = jac + 54 * (long long)f + (c - 9);
#pragma unroll
    for (int r = 0; r < 9; ++r) o[6 * r] = x[r];
  }
  // the symmetric part of S (the lanes' columns meet in LDS; a row's 16 lanes are in one wave)
  if (c < 9) {
#pragma unroll
    for (int r = 0; r < 9; ++r) sS[slot][r][c] = x[r];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (c < 9) {
    double* oc = cov + 81 * (long long)f + c;
#pragma unroll
    for (int r = 0; r < 9; ++r) oc[9 * r] = 0.5 * (x[r] + sS[slot][c][r]);
  }
}

__global__ __launch_bounds__(kImuBlock) void imu_linearize_kernel(
    const double* __restrict__ pre, const double* __restrict__ cov, const int* __restrict__ idx,
    int F, const double* __restrict__ poses, const double* __restrict__ vel, int P, double g0,
    double g1, double g2, double* __restrict__ H, double* __restrict__ bout,
    double* __restrict__ err, unsigned* __restrict__ flags) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= F) return;
  const int i = idx[2 * f], j = idx[2 * f + 1];
  if (i < 0 || i >= P || j < 0 || j >= P) {
    atomicOr(flags, kFlagBadIndex);
    return;
  }
  const double* p = pre + 16 * (long long)f;
  const double* Ti = poses + 12 * (long long)i;
  const double* Tj = poses + 12 * (long long)j;
  double Ri[3][3], Rj[3][3], ti[3], tj[3], vi[3], vj[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      Ri[r][c] = Ti[4 * r + c];
      Rj[r][c] = Tj[4 * r + c];
    }
    ti[r] = Ti[4 * r + 3];
    tj[r] = Tj[4 * r + 3];
    vi[r] = vel[3 * i + r];
    vj[r] = vel[3 * j + r];
  }
  const double dt = p[15];
  const double g[3] = {g0, g1, g2};
  // rotation residual: Log(dR^T Ri^T Rj)
  double M[3][3], Rij[3][3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) Rij[r][c] = Ri[0][r] * Rj[0][c] + Ri[1][r] * Rj[1][c] + Ri[2][r] * Rj[2][c];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      M[r][c] = p[r] * Rij[0][c] + p[3 + r] * Rij[1][c] + p[6 + r] * Rij[2][c];
  double res[9], Ji[3][3];
  so3_log_jrinv(M, res, Ji);
  double uv[3], up[3];  // Ri^T (vj - vi - g dt), Ri^T (tj - ti - vi dt - g dt^2 / 2)
  {
    double a[3], b[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      a[r] = vj[r] - vi[r] - g[r] * dt;
      b[r] = tj[r] - ti[r] - vi[r] * dt - 0.5 * g[r] * dt * dt;
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      uv[r] = Ri[0][r] * a[0] + Ri[1][r] * a[1] + Ri[2][r] * a[2];
      up[r] = Ri[0][r] * b[0] + Ri[1][r] * b[1] + Ri[2][r] * b[2];
      res[3 + r] = uv[r] - p[9 + r];
      res[6 + r] = up[r] - p[12 + r];
    }
  }
  // Jacobian 9 x 18 over [xi_i (omega, rho), v_i, xi_j (omega, rho), v_j]
  double J[9][18];
#pragma unroll
  for (int r = 0; r < 9; ++r)
#pragma unroll
    for (int c = 0; c < 18; ++c) J[r][c] = 0.0;
  double Kv[3][3], Kp[3][3];
  hat3(uv, Kv);
  hat3(up, Kp);
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      // -Jr^-1 Rj^T Ri = -Jr^-1 Rij^T
      J[r][c] = -(Ji[r][0] * Rij[c][0] + Ji[r][1] * Rij[c][1] + Ji[r][2] * Rij[c][2]);
      J[r][9 + c] = Ji[r][c];
      J[3 + r][c] = Kv[r][c];
      J[3 + r][6 + c] = -Ri[c][r];
      J[3 + r][15 + c] = Ri[c][r];
      J[6 + r][c] = Kp[r][c];
      J[6 + r][3 + c] = r == c ? -1.0 : 0.0;
      J[6 + r][6 + c] = -Ri[c][r] * dt;
      J[6 + r][12 + c] = Rij[r][c];
    }
  // whiten with the Cholesky factor L of the covariance (S = L L^T): solve L Y = [J | r]
  double L[9][9];
  const double* S = cov + 81 * (long long)f;
  bool pd = true;
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    double d = S[9 * c + c];
#pragma unroll
    for (int q = 0; q < c; ++q) d -= L[c][q] * L[c][q];
    if (!(d > 1e-13 * S[9 * c + c])) {  // not positive definite to working precision
      pd = false;
      d = 1.0;
    }
    const double lc = sqrt(d);
    L[c][c] = lc;
#pragma unroll
    for (int r = c + 1; r < 9; ++r) {
      double v = S[9 * r + c];
#pragma unroll
      for (int q = 0; q < c; ++q) v -= L[r][q] * L[c][q];
      L[r][c] = v / lc;
    }
  }
  if (!pd) atomicOr(flags, kFlagNonFinite);
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const double inv = 1.0 / L[r][r];
#pragma unroll
    for (int c = 0; c < 18; ++c) {
      double v = J[r][c];
#pragma unroll
      for (int q = 0; q < r; ++q) v -= L[r][q] * J[q][c];
      J[r][c] = v * inv;
    }
    double v = res[r];
#pragma unroll
    for (int q = 0; q < r; ++q) v -= L[r][q] * res[q];
    res[r] = v * inv;
  }
  double* Ho = H + 324 * (long long)f;
#pragma unroll
  for (int a = 0; a < 18; ++a)
#pragma unroll
    for (int c = 0; c < 18; ++c) {
      double v = 0.0;
#pragma unroll
      for (int r = 0; r < 9; ++r) v += J[r][a] * J[r][c];
      Ho[18 * a + c] = v;
    }
#pragma unroll
  for (int a = 0; a < 18; ++a) {
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < 9; ++r) v += J[r][a] * res[r];
    bout[18 * (long long)f + a] = v;
  }
  double e = 0.0;
#pragma unroll
  for (int r = 0; r < 9; ++r) e += res[r] * res[r];
  err[f] = e;
}

// Factor with bias states (the state of Eq. (1) holds the biases): the preintegrated values
// corrected to first order for the bias of state i (db = b_i - b0, b0 the preintegration's),
//   dR Exp(J_R,w db_w), dv + J_v db, dp + J_p db,
// the residual above with them, and the bias random walk b_j - b_i (covariance
// diag(sigma_ba^2, sigma_bw^2) dt): 15 residuals over 30 unknowns [xi_i, v_i, b_i, xi_j, v_j, b_j].
// Eight factors per block of 256 threads: a lane per factor forms the residual and the Jacobian's
// nonzero blocks in LDS while a lane per factor of another wave forms the Cholesky factor of the
// preintegration covariance in registers (with a block per factor that serial part was issued for
// one lane at a time, and 4,000 of them took 40 us); then a thread per column whitens [J | r], and a
// thread per column of H = J~^T J~ keeps its own column of J~ in registers; b = J~^T r~, e = |r~|^2.
constexpr int kImuBiasThreads = 256, kImuBiasFactors = 8;
__global__ __launch_bounds__(kImuBiasThreads) void imu_linearize_bias_kernel(
    const double* __restrict__ pre, const double* __restrict__ cov,
    const double* __restrict__ jac, const double* __restrict__ bias0,
    const int* __restrict__ idx, int F, const double* __restrict__ poses,
    const double* __restrict__ vel, const double* __restrict__ biases, int P, double g0,
    double g1, double g2, double qa, double qw, double* __restrict__ H,
    double* __restrict__ bout, double* __restrict__ err, unsigned* __restrict__ flags) {
  __shared__ double sJ[kImuBiasFactors][15][31];  // column 30: the residual
  __shared__ double sL[kImuBiasFactors][9][9];    // below the diagonal L, on it 1 / L[c][c]
  __shared__ double sw[kImuBiasFactors][6];
  __shared__ int ok_range[kImuBiasFactors], ok_val[kImuBiasFactors], ok_pd[kImuBiasFactors];
  const int f0 = blockIdx.x * kImuBiasFactors, t = threadIdx.x;
  for (int e = t; e < kImuBiasFactors * 15 * 31; e += kImuBiasThreads) (&sJ[0][0][0])[e] = 0.0;
  __syncthreads();
  if (t >= 64 && t < 64 + kImuBiasFactors && f0 + t - 64 < F) {
    const int u = t - 64;
    const double* S = cov + 81 * (long long)(f0 + u);
    double L[9][9];
    bool pd = true;
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      double d = S[9 * c + c];
#pragma unroll
      for (int q = 0; q < c; ++q) d -= L[c][q] * L[c][q];
      if (!(d > 1e-13 * S[9 * c + c])) {  // not positive definite to working precision
        pd = false;
        d = 1.0;
      }
      const double lc = sqrt(d), inv = 1.0 / lc;
      L[c][c] = lc;
#pragma unroll
      for (int r = c + 1; r < 9; ++r) {
        double v = S[9 * r + c];
#pragma unroll
        for (int q = 0; q < c; ++q) v -= L[r][q] * L[c][q];
        L[r][c] = v * inv;
      }
      sL[u][c][c] = inv;
    }
#pragma unroll
    for (int r = 0; r < 9; ++r)
#pragma unroll
      for (int c = 0; c < r; ++c) sL[u][r][c] = L[r][c];
    ok_pd[u] = pd ? 1 : 0;
  }
  if (t < kImuBiasFactors && f0 + t < F) {
    const int f = f0 + t;
    double (*J)[31] = sJ[t];
    double* wb = sw[t];
    int ok = 1;
    const int i = idx[2 * f], j = idx[2 * f + 1];
    if (i < 0 || i >= P || j < 0 || j >= P) {
      atomicOr(flags, kFlagBadIndex);
      ok_range[t] = 0;
    } else {
      ok_range[t] = 1;
      const double* p = pre + 16 * (long long)f;
      const double* Jb = jac + 54 * (long long)f;  // [9][6]
      const double* Ti = poses + 12 * (long long)i;
      const double* Tj = poses + 12 * (long long)j;
      double Ri[3][3], Rj[3][3], ti[3], tj[3], vi[3], vj[3], db[6];
      for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) {
          Ri[r][c] = Ti[4 * r + c];
          Rj[r][c] = Tj[4 * r + c];
        }
        ti[r] = Ti[4 * r + 3];
        tj[r] = Tj[4 * r + 3];
        vi[r] = vel[3 * i + r];
        vj[r] = vel[3 * j + r];
      }
      for (int k = 0; k < 6; ++k) db[k] = biases[6 * i + k] - bias0[6 * (long long)f + k];
      const double dt = p[15];
      const double g[3] = {g0, g1, g2};
      // the corrected preintegration
      double phi[3], Ephi[3][3], Jphi[3][3], dRc[3][3], dvc[3], dpc[3];
      for (int r = 0; r < 3; ++r)
        phi[r] = Jb[6 * r + 3] * db[3] + Jb[6 * r + 4] * db[4] + Jb[6 * r + 5] * db[5];
      so3_exp_jr(phi, Ephi, Jphi);
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
          dRc[r][c] = p[3 * r] * Ephi[0][c] + p[3 * r + 1] * Ephi[1][c] + p[3 * r + 2] * Ephi[2][c];
      for (int r = 0; r < 3; ++r) {
        double sv = p[9 + r], sp = p[12 + r];
        for (int k = 0; k < 6; ++k) {
          sv += Jb[6 * (3 + r) + k] * db[k];
          sp += Jb[6 * (6 + r) + k] * db[k];
        }
        dvc[r] = sv;
        dpc[r] = sp;
      }
      // rotation residual Log(dRc^T Ri^T Rj) and its right Jacobian's inverse
      double Rij[3][3], M[3][3], rR[3], Ji[3][3];
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
          Rij[r][c] = Ri[0][r] * Rj[0][c] + Ri[1][r] * Rj[1][c] + Ri[2][r] * Rj[2][c];
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
          M[r][c] = dRc[0][r] * Rij[0][c] + dRc[1][r] * Rij[1][c] + dRc[2][r] * Rij[2][c];
      so3_log_jrinv(M, rR, Ji);
      double uv[3], up[3];
      {
        double a[3], b[3];
        for (int r = 0; r < 3; ++r) {
          a[r] = vj[r] - vi[r] - g[r] * dt;
          b[r] = tj[r] - ti[r] - vi[r] * dt - 0.5 * g[r] * dt * dt;
        }
        for (int r = 0; r < 3; ++r) {
          uv[r] = Ri[0][r] * a[0] + Ri[1][r] * a[1] + Ri[2][r] * a[2];
          up[r] = Ri[0][r] * b[0] + Ri[1][r] * b[1] + Ri[2][r] * b[2];
        }
      }
      for (int r = 0; r < 3; ++r) {
        J[r][30] = rR[r];
        J[3 + r][30] = uv[r] - dvc[r];
        J[6 + r][30] = up[r] - dpc[r];
      }
      for (int k = 0; k < 6; ++k) J[9 + k][30] = biases[6 * j + k] - biases[6 * i + k];
      // the gyro-bias column of the rotation: -J_r^-1(rR) Exp(rR)^T J_r(phi) J_R,w, Exp(rR) = M
      double G[3][3], Q[3][3];
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
          G[r][c] = Jphi[r][0] * Jb[3 + c] + Jphi[r][1] * Jb[6 + 3 + c] +
                    Jphi[r][2] * Jb[12 + 3 + c];
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
          Q[r][c] = M[0][r] * G[0][c] + M[1][r] * G[1][c] + M[2][r] * G[2][c];
      double Kv[3][3], Kp[3][3];
      hat3(uv, Kv);
      hat3(up, Kp);
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
          J[r][c] = -(Ji[r][0] * Rij[c][0] + Ji[r][1] * Rij[c][1] + Ji[r][2] * Rij[c][2]);
          J[r][15 + c] = Ji[r][c];
          J[r][12 + c] = -(Ji[r][0] * Q[0][c] + Ji[r][1] * Q[1][c] + Ji[r][2] * Q[2][c]);
          J[3 + r][c] = Kv[r][c];
          J[3 + r][6 + c] = -Ri[c][r];
          J[3 + r][21 + c] = Ri[c][r];
          J[6 + r][c] = Kp[r][c];
          J[6 + r][3 + c] = r == c ? -1.0 : 0.0;
          J[6 + r][6 + c] = -Ri[c][r] * dt;
          J[6 + r][18 + c] = Rij[r][c];
        }
      for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 6; ++k) {
          J[3 + r][9 + k] = -Jb[6 * (3 + r) + k];
          J[6 + r][9 + k] = -Jb[6 * (6 + r) + k];
        }
      for (int k = 0; k < 6; ++k) {
        J[9 + k][9 + k] = -1.0;
        J[9 + k][24 + k] = 1.0;
        const double q = (k < 3 ? qa : qw) * dt;
        wb[k] = 1.0 / sqrt(q);
        if (!(q > 0.0) || !isfinite(q)) ok = 0;
      }
    }
    ok_val[t] = ok;
  }
  __syncthreads();
  if (t < kImuBiasFactors && f0 + t < F && ok_range[t] && !(ok_val[t] && ok_pd[t]))
    atomicOr(flags, kFlagNonFinite);
  // whiten the columns of [J | r]: L^-1 for the preintegration rows, 1 / sqrt(q dt) for the walk
  if (t < kImuBiasFactors * 31) {
    const int u = t / 31, c = t - 31 * u;
    if (f0 + u < F && ok_range[u] && ok_val[u] && ok_pd[u]) {
      double y[9];
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        double v = sJ[u][r][c];
#pragma unroll
        for (int q = 0; q < r; ++q) v -= sL[u][r][q] * y[q];
        y[r] = v * sL[u][r][r];
      }
#pragma unroll
      for (int r = 0; r < 9; ++r) sJ[u][r][c] = y[r];
#pragma unroll
      for (int r = 0; r < 6; ++r) sJ[u][9 + r][c] *= sw[u][r];
    }
  }
  __syncthreads();
  if (t < kImuBiasFactors * 30) {
    const int u = t / 30, c = t - 30 * u;
    const int f = f0 + u;
    if (f >= F || !(ok_range[u] && ok_val[u] && ok_pd[u])) return;
    double col[15];
#pragma unroll
    for (int r = 0; r < 15; ++r) col[r] = sJ[u][r][c];
    double* Ho = H + 900 * (long long)f + c;
    for (int a = 0; a < 30; ++a) {  // column c of row a: a wave's lanes write whole rows
      double v = 0.0;
#pragma unroll
      for (int r = 0; r < 15; ++r) v += sJ[u][r][a] * col[r];
      Ho[30 * a] = v;
    }
    double v = 0.0, e = 0.0;
#pragma unroll
    for (int r = 0; r < 15; ++r) {
      v += col[r] * sJ[u][r][30];
      e += sJ[u][r][30] * sJ[u][r][30];
    }
    bout[30 * (long long)f + c] = v;
    if (c == 0) err[f] = e;
  }
}

}  // namespace

void launch_imu_preintegrate(const double* imu, int64_t m, const int64_t* seg, int F,
                             const double* bias,
                             double sigma_g, double sigma_a, double* pre, double* cov,
                             double* jac, unsigned* flags, hipStream_t s) {
  if (F <= 0) return;
  const unsigned grid = (unsigned)(((long long)F * kImuLanes + kImuBlock - 1) / kImuBlock);
  imu_preintegrate_kernel<<<grid, kImuBlock, 0, s>>>(
      imu, (long long)m, reinterpret_cast<const long long*>(seg), F, bias, sigma_g * sigma_g,
      sigma_a * sigma_a, pre, cov, jac, flags);
}

void launch_imu_linearize_bias(const double* pre, const double* cov, const double* jac,
                               const double* bias0, const int32_t* idx, int F,
                               const double* poses, const double* vel, const double* biases,
                               int P, const double g[3], double sigma_ba, double sigma_bw,
                               double* H, double* b, double* err, unsigned* flags,
                               hipStream_t s) {
  if (F <= 0) return;
  imu_linearize_bias_kernel<<<(F + kImuBiasFactors - 1) / kImuBiasFactors, kImuBiasThreads, 0, s>>>(
      pre, cov, jac, bias0, idx, F, poses, vel, biases, P, g[0], g[1], g[2],
      sigma_ba * sigma_ba, sigma_bw * sigma_bw, H, b, err, flags);
}

void launch_imu_linearize(const double* pre, const double* cov, const int32_t* idx, int F,
                          const double* poses, const double* vel, int P, const double g[3],
                          double* H, double* b, double* err, unsigned* flags, hipStream_t s) {
  if (F <= 0) return;
  imu_linearize_kernel<<<(F + kImuBlock - 1) / kImuBlock, kImuBlock, 0, s>>>(
      pre, cov, idx, F, poses, vel, P, g[0], g[1], g[2], H, b, err, flags);
}

}  // namespace vgicp
