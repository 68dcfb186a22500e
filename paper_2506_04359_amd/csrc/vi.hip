// Visual-inertial window solve (paper Sec. 2.2, "Visual-Inertial", Eq. 9).
//
// The state of keyframe i is S_i = [T_i, v_i, b^a_i, b^w_i]; consecutive
// states are tied by an IMU factor built from the on-manifold preintegration
// of the samples between them (the model of Forster et al. 2017 that the
// paper cites).  The visual part of the window solve is unchanged; per LM
// attempt and window this file adds
//   k_vi_fac   one workgroup per IMU factor at the current state: residual,
//              Jacobian, J^T Lambda J and J^T Lambda r (FP64) into the
//              factor's record;
//   k_vi_lin   the pose-pose terms added into the summed reduced system and
//              the elimination of the extra variables y = (v, b^a, b^w) onto
//              the poses: A = H_yy + damping is block tridiagonal (9x9
//              blocks); with X = A^-1 H_yx and z = A^-1 g_y,
//                  S <- S - H_xy X,   rhs <- rhs + H_xy z,
//              so the reduced camera system keeps its size and the existing
//              Cholesky solves it;
//   k_vi_cand  after the poses' step dx: dy = -z - X dx, the candidate
//              velocities and biases, and the IMU cost at the candidate.
// Everything here is FP64 (a window has few IMU factors; their information
// matrices span many orders of magnitude).
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>
#include <type_traits>

#include "device.hpp"
#include "geometry.hpp"
#include "vi.hpp"

namespace ba {
namespace {

// ---- SO(3) on 3x3 row-major matrices
__device__ void skew3(const double* v, double* K) {
  K[0] = 0.0;
  K[1] = -v[2];
  K[2] = v[1];
  K[3] = v[2];
  K[4] = 0.0;
  K[5] = -v[0];
  K[6] = -v[1];
  K[7] = v[0];
  K[8] = 0.0;
}

__device__ void mul33(const double* A, const double* B, double* C) {
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) C[3 * a + b] = A[3 * a] * B[b] + A[3 * a + 1] * B[3 + b] + A[3 * a + 2] * B[6 + b];
}

__device__ void mul33t(const double* A, const double* B, double* C) {   // A^T B
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) C[3 * a + b] = A[a] * B[b] + A[3 + a] * B[3 + b] + A[6 + a] * B[6 + b];
}

__device__ void mul3t3(const double* A, const double* B, double* C) {   // A B^T
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      C[3 * a + b] = A[3 * a] * B[3 * b] + A[3 * a + 1] * B[3 * b + 1] + A[3 * a + 2] * B[3 * b + 2];
}

__device__ void mv3(const double* A, const double* x, double* y) {
  for (int a = 0; a < 3; ++a) y[a] = A[3 * a] * x[0] + A[3 * a + 1] * x[1] + A[3 * a + 2] * x[2];
}

__device__ void mtv3(const double* A, const double* x, double* y) {   // A^T x
  for (int a = 0; a < 3; ++a) y[a] = A[a] * x[0] + A[3 + a] * x[1] + A[6 + a] * x[2];
}

// sin(th)/th, (1 - cos th)/th^2, (th - sin th)/th^3 (power series below th = 1)
__device__ void so3_coeffs(double th2, double& A, double& B, double& C) {
  if (th2 < 1.0) {
    double a = 1.0, b = 1.0, c = 1.0;
    for (int k = 8; k >= 0; --k) {
      const double n = 2.0 * k;
      a = fma(-th2 * (1.0 / ((n + 2.0) * (n + 3.0))), a, 1.0);
      b = fma(-th2 * (1.0 / ((n + 3.0) * (n + 4.0))), b, 1.0);
      c = fma(-th2 * (1.0 / ((n + 4.0) * (n + 5.0))), c, 1.0);
    }
    A = a;
    B = 0.5 * b;
    C = c / 6.0;
  } else {
    const double th = sqrt(th2);
    A = sin(th) / th;
    const double s = sin(0.5 * th);
    B = 2.0 * s * s / th2;
    C = (th - sin(th)) / (th2 * th);
  }
}

// Exp(phi) and the right Jacobian J_r(phi) = I - B K + C K^2.
__device__ void exp_so3_jr(const double* phi, double* R, double* Jr) {
  const double th2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
  double A, B, C;
  so3_coeffs(th2, A, B, C);
  double K[9], K2[9];
  skew3(phi, K);
  mul33(K, K, K2);
  for (int k = 0; k < 9; ++k) {
    const double I = (k % 4 == 0) ? 1.0 : 0.0;
    R[k] = I + A * K[k] + B * K2[k];
    if (Jr) Jr[k] = I - B * K[k] + C * K2[k];
  }
}

// Log of a rotation (theta from atan2 of the antisymmetric and trace parts;
// the axis from the symmetric part near theta = pi).
__device__ void log_so3_33(const double* R, double* phi) {
  const double v[3] = {0.5 * (R[7] - R[5]), 0.5 * (R[2] - R[6]), 0.5 * (R[3] - R[1])};
  double c = 0.5 * (R[0] + R[4] + R[8] - 1.0);
  c = fmin(1.0, fmax(-1.0, c));
  const double s = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  const double th = atan2(s, c);
  if (c > -0.999) {
    const double t2 = th * th;
    const double f = th < 1e-3 ? 1.0 + t2 * (1.0 / 6.0 + t2 * (7.0 / 360.0)) : th / s;
    for (int k = 0; k < 3; ++k) phi[k] = f * v[k];
    return;
  }
  const double Md[3] = {R[0] - c, R[4] - c, R[8] - c};
  int k = 0;
  if (Md[1] > Md[k]) k = 1;
  if (Md[2] > Md[k]) k = 2;
  const double ic = 1.0 / (1.0 - c);
  double a[3];
  a[k] = sqrt(fmax(Md[k] * ic, 0.0));
  const double ia = 1.0 / a[k];
  for (int m = 0; m < 3; ++m)
    if (m != k) a[m] = 0.5 * (R[3 * m + k] + R[3 * k + m]) * ic * ia;
  const double sg = (a[0] * v[0] + a[1] * v[1] + a[2] * v[2]) < 0.0 ? -1.0 : 1.0;
  for (int m = 0; m < 3; ++m) phi[m] = sg * th * a[m];
}

// J_r(phi)^-1 = I + K / 2 + d K^2, d = 1/th^2 - cot(th/2) / (2 th)
__device__ void jr_inv(const double* phi, double* Ji) {
  const double t2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
  double d;
  if (t2 < 1e-2) {
    d = 1.0 / 12.0 + t2 * (1.0 / 720.0 + t2 * (1.0 / 30240.0 + t2 * (1.0 / 1209600.0)));
  } else {
    const double th = sqrt(t2);
    d = 1.0 / t2 - cos(0.5 * th) / (sin(0.5 * th) * 2.0 * th);
  }
  double K[9], K2[9];
  skew3(phi, K);
  mul33(K, K, K2);
  for (int k = 0; k < 9; ++k) Ji[k] = ((k % 4 == 0) ? 1.0 : 0.0) + 0.5 * K[k] + d * K2[k];
}

// In-place Cholesky A = L L^T of an n x n row-major matrix (lower part
// written); false on a non-positive or non-finite pivot.
__device__ bool chol_n(double* A, int n) {
  for (int j = 0; j < n; ++j) {
    double d = A[n * j + j];
    for (int k = 0; k < j; ++k) d -= A[n * j + k] * A[n * j + k];
    if (!(d > 0.0) || !isfinite(d)) return false;
    const double l = sqrt(d);
    A[n * j + j] = l;
    const double il = 1.0 / l;
    for (int i = j + 1; i < n; ++i) {
      double v = A[n * i + j];
      for (int k = 0; k < j; ++k) v -= A[n * i + k] * A[n * j + k];
      A[n * i + j] = v * il;
    }
  }
  return true;
}

// y = L^-1 x and x = L^-T y for a Cholesky factor in the lower part of L (n x n)
__device__ void lsolve(const double* L, int n, double* x) {
  for (int i = 0; i < n; ++i) {
    double v = x[i];
    for (int k = 0; k < i; ++k) v -= L[n * i + k] * x[k];
    x[i] = v / L[n * i + i];
  }
}

__device__ void ltsolve(const double* L, int n, double* x) {
  for (int i = n - 1; i >= 0; --i) {
    double v = x[i];
    for (int k = i + 1; k < n; ++k) v -= L[n * k + i] * x[k];
    x[i] = v / L[n * i + i];
  }
}

// Residual (15) of the factor between states i and j and, with kJac, its
// Jacobian: 15 x 30 row-major, columns (rho_i, phi_i, v_i, b^a_i, b^w_i,
// rho_j, phi_j, v_j, b^a_j, b^w_j); only the non-zero entries are written (J
// must hold zeros).  pose: 3x4 base-from-world, st: v, b^a, b^w.
template <bool kJac>
__device__ void imu_factor(const double* Pi, const double* si, const double* Pj, const double* sj,
                           const double* pre, const double* g, double* r, double* J) {
  const double Ri[9] = {Pi[0], Pi[1], Pi[2], Pi[4], Pi[5], Pi[6], Pi[8], Pi[9], Pi[10]};
  const double Rj[9] = {Pj[0], Pj[1], Pj[2], Pj[4], Pj[5], Pj[6], Pj[8], Pj[9], Pj[10]};
  const double ti[3] = {Pi[3], Pi[7], Pi[11]}, tj[3] = {Pj[3], Pj[7], Pj[11]};
  double pi[3], pj[3];
  mtv3(Ri, ti, pi);
  mtv3(Rj, tj, pj);
  for (int k = 0; k < 3; ++k) {
    pi[k] = -pi[k];
    pj[k] = -pj[k];
  }
  const double* dR = pre + kPreDR;
  const double* JRg = pre + kPreJRg;
  double dbg[3], dba[3];
  for (int k = 0; k < 3; ++k) {
    dbg[k] = si[6 + k] - pre[kPreBg + k];
    dba[k] = si[3 + k] - pre[kPreBa + k];
  }
  double u[3], Eu[9], Jru[9], dRc[9];
  mv3(JRg, dbg, u);
  exp_so3_jr(u, Eu, Jru);
  mul33(dR, Eu, dRc);
  double RiRjT[9], E[9];
  mul3t3(Ri, Rj, RiRjT);          // R_i R_j^T
  mul33t(dRc, RiRjT, E);          // dRc^T R_i R_j^T
  double rR[3];
  log_so3_33(E, rR);
  const double dT = pre[kPreDT];
  double wv[3], wp[3];
  for (int k = 0; k < 3; ++k) {
    wv[k] = sj[k] - si[k] - g[k] * dT;
    wp[k] = pj[k] - pi[k] - si[k] * dT - 0.5 * g[k] * dT * dT;
  }
  double Riwv[3], Riwp[3];
  mv3(Ri, wv, Riwv);
  mv3(Ri, wp, Riwp);
  const double* Jvg = pre + kPreJvg;
  const double* Jva = pre + kPreJva;
  const double* Jpg = pre + kPreJpg;
  const double* Jpa = pre + kPreJpa;
  for (int a = 0; a < 3; ++a) {
    double cv = pre[kPreDv + a], cp = pre[kPreDp + a];
    for (int b = 0; b < 3; ++b) {
      cv += Jvg[3 * a + b] * dbg[b] + Jva[3 * a + b] * dba[b];
      cp += Jpg[3 * a + b] * dbg[b] + Jpa[3 * a + b] * dba[b];
    }
    r[a] = rR[a];
    r[3 + a] = Riwv[a] - cv;
    r[6 + a] = Riwp[a] - cp;
    r[9 + a] = sj[3 + a] - si[3 + a];
    r[12 + a] = sj[6 + a] - si[6 + a];
  }
  if (!kJac) return;
  double Jri[9];
  jr_inv(rR, Jri);
  double RjRiT[9], T1[9], T2[9], T3[9];
  mul3t3(Rj, Ri, RjRiT);
  mul33(Jri, RjRiT, T1);          // dr_R/dphi_i
  mul33t(E, Jru, T2);             // E^T J_r(u)
  mul33(T2, JRg, T3);             // E^T J_r(u) J_Rg
  double T4[9];
  mul33(Jri, T3, T4);
  double Kv[9], Kp[9];
  skew3(Riwv, Kv);
  skew3(Riwp, Kp);
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) {
      const int k = 3 * a + b;
      const double I = a == b ? 1.0 : 0.0;
      // r_R
      J[30 * a + 3 + b] = T1[k];
      J[30 * a + 12 + b] = -T4[k];
      J[30 * a + 18 + b] = -Jri[k];
      // r_v
      J[30 * (3 + a) + 3 + b] = -Kv[k];
      J[30 * (3 + a) + 6 + b] = -Ri[k];
      J[30 * (3 + a) + 9 + b] = -Jva[k];
      J[30 * (3 + a) + 12 + b] = -Jvg[k];
      J[30 * (3 + a) + 21 + b] = Ri[k];
      // r_p
      J[30 * (6 + a) + 0 + b] = I;
      J[30 * (6 + a) + 3 + b] = -Kp[k];
      J[30 * (6 + a) + 6 + b] = -Ri[k] * dT;
      J[30 * (6 + a) + 9 + b] = -Jpa[k];
      J[30 * (6 + a) + 12 + b] = -Jpg[k];
      J[30 * (6 + a) + 15 + b] = -RiRjT[k];
      // bias random walk
      if (a == b) {
        J[30 * (9 + a) + 9 + b] = -1.0;
        J[30 * (9 + a) + 24 + b] = 1.0;
        J[30 * (12 + a) + 12 + b] = -1.0;
        J[30 * (12 + a) + 27 + b] = 1.0;
      }
    }
}

// A double of lane L of the own four lanes.
template <int L>
__device__ __forceinline__ double quad_value(double v) {
  const long long b = __double_as_longlong(v);
  constexpr int ctrl = L * 0x55;   // quad_perm L, L, L, L
  const unsigned lo = __builtin_amdgcn_mov_dpp((int)b, ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), ctrl, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | lo);
}

// LDS of one wave: its accesses above done before those below.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ double imu_cost1(const double* r, const double* Info) {
  double c = 0.0;
  for (int a = 0; a < 15; ++a) {
    double v = 0.0;
    for (int b = 0; b < 15; ++b) v += Info[15 * a + b] * r[b];
    c += r[a] * v;
  }
  return 0.5 * c;
}

}  // namespace

// ---------------------------------------------------------------------------
// preintegration: one workgroup per factor, samples in time order
// ---------------------------------------------------------------------------

// Four chains run over a factor's samples: the rotation dR, the 9x9 covariance, the
// gyroscope bias' Jacobians, and those of the accelerometer bias with the velocity and
// position.  A thread per factor took 3 us a sample (148 us for nine factors of 50
// samples): about a thousand instructions in one lane.  Here what a sample needs by itself (Exp,
// J_r, the noise products) is worked out a sample per lane, the rotation chain by three
// lanes, and the other chains each by a wave of its own, an entry's (or a row's)
// products per lane: 27 us.  Every entry keeps its sums' order, the fused products
// written out where the order of the terms leaves the choice.
constexpr int kPreThreads = 256, kPreSamples = 64;   // samples staged at a time
constexpr int kPsE = 0, kPsJr = 9, kPsGG = 18, kPsR = 27, kPsX = 36, kPsB = 45, kPsAA = 54, kPsA = 63, kPsRa = 66,
              kPsRec = 69;   // a sample's record: Exp, J_r, J_r J_r^T, dR, dR [a]x, -dR [a]x dt, dR dR^T, a, dR a
// odd, so that the lanes of a wave (a sample each) meet no bank twice in a row
static_assert(kPsRec % 2 == 1, "record stride");

// a0 b0 + a1 b1 + a2 b2
__device__ __forceinline__ double dot3(double a0, double b0, double a1, double b1, double a2, double b2) {
  return fma(a2, b2, fma(a0, b0, a1 * b1));
}

__global__ __launch_bounds__(kPreThreads) void k_vi_preint(const int32_t* sample_begin, const double* gyro,
                                                           const double* accel, double dt,
                                                           const double* bias_bar, double sg, double sa, double sbg,
                                                           double sba, double* out) {
  __shared__ double sS[kPreSamples * kPsRec];
  __shared__ double sP[81];   // covariance of the errors (dphi, dv, dp): 3x3 blocks P_ij, i <= j, 9 (3 i + j)
  const int f = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  double* pre = out + (size_t)kPreStride * f;
  const double ba[3] = {bias_bar[6 * f], bias_bar[6 * f + 1], bias_bar[6 * f + 2]};
  const double bg[3] = {bias_bar[6 * f + 3], bias_bar[6 * f + 4], bias_bar[6 * f + 5]};
  const double qg = sg * sg / dt, qa = sa * sa / dt, h = 0.5 * dt;
  const int s0 = sample_begin[f], s1 = sample_begin[f + 1];
  if (tid < 81) sP[tid] = 0.0;
  // wave 0: lanes 0-2 a row of dR in its first phase; then lane 4 (3 i + x) + j row x of
  // the blocks (A P)_ij and, i <= j, P_ij
  double dR[3] = {lane == 0 ? 1.0 : 0.0, lane == 1 ? 1.0 : 0.0, lane == 2 ? 1.0 : 0.0};
  const int pj = lane & 3, pi = (lane >> 2) / 3, px = (lane >> 2) % 3;
  const bool pact = pj < 3 && pi < 3;
  // wave 1, lanes 0-2: a column of J_Rg, J_vg, J_pg; wave 2, lanes 0-8: an entry of J_va,
  // J_pa; wave 3, lanes 0-2: an entry of dv, dp
  double J[3] = {}, Jv[3] = {}, Jp[3] = {};
  for (int base = s0; base < s1; base += kPreSamples) {
    const int ns = min(kPreSamples, s1 - base);
    if (tid < ns) {
      const int s = base + tid;
      double* R = sS + kPsRec * tid;
      double w[3], a[3], Ek[9], Jr[9];
      for (int k = 0; k < 3; ++k) {
        w[k] = (gyro[3 * s + k] - bg[k]) * dt;
        a[k] = accel[3 * s + k] - ba[k];
      }
      exp_so3_jr(w, Ek, Jr);
      for (int k = 0; k < 9; ++k) {
        R[kPsE + k] = Ek[k];
        R[kPsJr + k] = Jr[k];
      }
      for (int k = 0; k < 3; ++k) R[kPsA + k] = a[k];
      for (int x = 0; x < 3; ++x)
        for (int y = 0; y < 3; ++y) {
          double gg = 0.0;
          for (int k = 0; k < 3; ++k) gg += Jr[3 * x + k] * Jr[3 * y + k];
          R[kPsGG + 3 * x + y] = gg;
        }
    }
    __syncthreads();
    if (tid < 3) {   // dR before each sample
      double E[9];
      for (int k = 0; k < 9; ++k) E[k] = sS[kPsE + k];
      for (int s = 0; s < ns; ++s) {
        double* R = sS + kPsRec * s;
        const double* Rn = sS + kPsRec * min(s + 1, ns - 1);
        double En[9];
        for (int k = 0; k < 9; ++k) En[k] = Rn[kPsE + k];
        for (int k = 0; k < 3; ++k) R[kPsR + 3 * tid + k] = dR[k];
        double nR[3];
        for (int k = 0; k < 3; ++k) nR[k] = dot3(dR[0], E[k], dR[1], E[3 + k], dR[2], E[6 + k]);
        for (int k = 0; k < 3; ++k) dR[k] = nR[k];
        for (int k = 0; k < 9; ++k) E[k] = En[k];
      }
    }
    __syncthreads();
    if (tid < ns) {
      double* R = sS + kPsRec * tid;
      double r[9], a[3], Ax[9], X[9], Ra[3];
      for (int k = 0; k < 9; ++k) r[k] = R[kPsR + k];
      for (int k = 0; k < 3; ++k) a[k] = R[kPsA + k];
      skew3(a, Ax);
      mul33(r, Ax, X);
      for (int k = 0; k < 3; ++k) Ra[k] = dot3(r[3 * k], a[0], r[3 * k + 1], a[1], r[3 * k + 2], a[2]);
      for (int k = 0; k < 9; ++k) {
        R[kPsX + k] = X[k];
        R[kPsB + k] = -X[k] * dt;
      }
      for (int k = 0; k < 3; ++k) R[kPsRa + k] = Ra[k];
      for (int x = 0; x < 3; ++x)
        for (int y = 0; y < 3; ++y) {
          double aa = 0.0;
          for (int k = 0; k < 3; ++k) aa += r[3 * x + k] * r[3 * y + k];
          R[kPsAA + 3 * x + y] = aa;
        }
    }
    __syncthreads();
    if (wave == 0) {
      // P <- A P A^T + noise with A = [[E^T, 0, 0], [B, I, 0], [B dt/2, dt I, I]] and
      // B = -dR [a]x dt: T = A P, then T A^T.  Row x of T_ij is the products with block
      // row 0 of P, plus rows of block rows 1 and 2; P_ij's are products with T_i0 (the
      // first lane of the four), plus rows of T_i1 and T_ij.
      const int i = pact ? pi : 0, j = pact ? pj : 0, x = px;
      // row x of P_1j and P_2j (a column of the block above the diagonal)
      const int a1 = j >= 1 ? 9 * (3 + j) + 3 * x : 9 * 1 + x, t1 = j >= 1 ? 1 : 3;
      const int a2 = j == 2 ? 9 * 8 + 3 * x : 9 * (3 * j + 2) + x, t2 = j == 2 ? 1 : 3;
      // the sample's coefficients: q of T, c of P, the noise term
      const int aq = i == 0 ? kPsE + x : kPsB + 3 * x, tq = i == 0 ? 3 : 1;
      const int ac = j == 0 ? kPsE : kPsB, tm = j == 0 ? 3 : 1, tb = j == 0 ? 1 : 3;
      const int an = (i == 0 ? kPsGG : kPsAA) + 3 * x;
      const bool noise = (i == 0 && j == 0) || i >= 1;
      const double cn = i == 0   ? qg * dt * dt
                        : j == 1 ? qa * dt * dt
                        : i == 1 ? qa * 0.5 * dt * dt * dt
                                 : qa * 0.25 * dt * dt * dt * dt;
      double q[3], c[9], n[3];
      auto coef = [&](int s, double (&qq)[3], double (&cc)[9], double (&nn)[3]) {
        const double* R = sS + kPsRec * s;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          qq[m] = R[aq + tq * m];
          nn[m] = R[an + m];
#pragma unroll
          for (int b = 0; b < 3; ++b) cc[3 * m + b] = R[ac + tm * m + tb * b];
        }
      };
      coef(0, q, c, n);
      for (int s = 0; s < ns; ++s) {
        double p0[9], p1[3], p2[3];
#pragma unroll
        for (int k = 0; k < 9; ++k) p0[k] = sP[9 * j + k];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          p1[b] = sP[a1 + t1 * b];
          p2[b] = sP[a2 + t2 * b];
        }
        double qn[3], cc[9], nn[3];
        coef(min(s + 1, ns - 1), qn, cc, nn);
        double T[3], T0[3], T1[3], P[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const double v = dot3(q[0], p0[b], q[1], p0[3 + b], q[2], p0[6 + b]);
          const double v2 = fma(h, v, dt * p1[b]) + p2[b];
          T[b] = i == 0 ? v : i == 1 ? v + p1[b] : v2;
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          T0[b] = quad_value<0>(T[b]);
          T1[b] = quad_value<1>(T[b]);
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const double v = dot3(T0[0], c[b], T0[1], c[3 + b], T0[2], c[6 + b]);
          const double v2 = fma(h, v, dt * T1[b]) + T[b];
          P[b] = j == 0 ? v : j == 1 ? v + T[b] : v2;
          if (noise) P[b] = fma(cn, n[b], P[b]);
        }
        wave_fence();   // the reads of sP above
        if (pact && i <= j)
#pragma unroll
          for (int b = 0; b < 3; ++b) sP[9 * (3 * i + j) + 3 * x + b] = P[b];
        wave_fence();
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          q[m] = qn[m];
          n[m] = nn[m];
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) c[k] = cc[k];
      }
    } else if (wave == 1) {
      const int b = min(lane, 2);
      for (int s = 0; s < ns; ++s) {
        const double* R = sS + kPsRec * s;
        double nJ[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const double m1 = dot3(R[kPsX + 3 * a], J[0], R[kPsX + 3 * a + 1], J[1], R[kPsX + 3 * a + 2], J[2]);
          const double et = dot3(R[kPsE + a], J[0], R[kPsE + 3 + a], J[1], R[kPsE + 6 + a], J[2]);
          Jp[a] += fma(Jv[a], dt, -(0.5 * m1 * dt * dt));
          Jv[a] = fma(-m1, dt, Jv[a]);
          nJ[a] = fma(-R[kPsJr + 3 * a + b], dt, et);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) J[a] = nJ[a];
      }
    } else if (wave == 2) {
      const int k = min(lane, 8);
#pragma unroll 4
      for (int s = 0; s < ns; ++s) {
        const double r = sS[kPsRec * s + kPsR + k];
        Jp[0] += fma(Jv[0], dt, -(0.5 * r * dt * dt));
        Jv[0] = fma(-r, dt, Jv[0]);
      }
    } else {
      const int k = min(lane, 2);
#pragma unroll 4
      for (int s = 0; s < ns; ++s) {
        const double r = sS[kPsRec * s + kPsRa + k];
        Jp[0] += fma(Jv[0], dt, 0.5 * r * dt * dt);
        Jv[0] = fma(r, dt, Jv[0]);
      }
    }
    __syncthreads();
  }
  const double dT = dt * (s1 - s0);
  double* Info = pre + kPreInfo;
  if (wave == 0) {
    if (lane < 3)
      for (int k = 0; k < 3; ++k) pre[kPreDR + 3 * lane + k] = dR[k];
  } else if (wave == 1) {
    if (lane < 3)
      for (int a = 0; a < 3; ++a) {
        pre[kPreJRg + 3 * a + lane] = J[a];
        pre[kPreJvg + 3 * a + lane] = Jv[a];
        pre[kPreJpg + 3 * a + lane] = Jp[a];
      }
  } else if (wave == 2) {
    if (lane < 9) {
      pre[kPreJva + lane] = Jv[0];
      pre[kPreJpa + lane] = Jp[0];
    }
  } else {
    if (lane < 3) {
      pre[kPreDv + lane] = Jv[0];
      pre[kPreDp + lane] = Jp[0];
      pre[kPreBa + lane] = ba[lane];
      pre[kPreBg + lane] = bg[lane];
    }
    if (lane == 0) pre[kPreDT] = dT;
  }
  // information: the inverse of the 9x9 covariance (Cholesky, a column per lane), the
  // bias random walk 1 / (sigma^2 dT).  One sample's covariance has rank 6 (the
  // same accelerometer noise moves velocity and position), so an interval of
  // fewer than two samples gets NaN information.
  for (int k = tid; k < 225; k += kPreThreads) {
    const int r = k / 15, c = k % 15;
    if (r < 9 && c < 9) continue;
    double v = 0.0;
    if (r == c) v = r < 12 ? 1.0 / (sba * sba * dT) : 1.0 / (sbg * sbg * dT);
    Info[k] = v;
  }
  if (tid < 9) {
    double cov[81];
#pragma unroll
    for (int r = 0; r < 9; ++r)
#pragma unroll
      for (int c = 0; c < 9; ++c)
        cov[9 * r + c] = r / 3 <= c / 3 ? sP[9 * (3 * (r / 3) + c / 3) + 3 * (r % 3) + c % 3]
                                        : sP[9 * (3 * (c / 3) + r / 3) + 3 * (c % 3) + r % 3];
    const bool ok = s1 - s0 >= 2 && chol_n(cov, 9);
    double e[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) e[k] = k == tid ? 1.0 : 0.0;
    if (ok) {
      lsolve(cov, 9, e);
      ltsolve(cov, 9, e);
    } else {
      for (int k = 0; k < 9; ++k) e[k] = __builtin_nan("");
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) Info[15 * k + tid] = e[k];
  }
}

// The same for many factors, one thread each: no lane idles.
__global__ __launch_bounds__(64) void k_vi_preint_many(int n_factors, const int32_t* sample_begin,
                                                       const double* gyro, const double* accel, double dt,
                                                       const double* bias_bar, double sg, double sa, double sbg,
                                                       double sba, double* out) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= n_factors) return;
  double* pre = out + (size_t)kPreStride * f;
  const double ba[3] = {bias_bar[6 * f], bias_bar[6 * f + 1], bias_bar[6 * f + 2]};
  const double bg[3] = {bias_bar[6 * f + 3], bias_bar[6 * f + 4], bias_bar[6 * f + 5]};
  double dR[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, dv[3] = {0, 0, 0}, dp[3] = {0, 0, 0};
  double JRg[9] = {}, Jvg[9] = {}, Jva[9] = {}, Jpg[9] = {}, Jpa[9] = {};
  // covariance of the errors (dphi, dv, dp) in 3x3 blocks P_ij, i <= j
  double P00[9] = {}, P01[9] = {}, P02[9] = {}, P11[9] = {}, P12[9] = {}, P22[9] = {};
  const double qg = sg * sg / dt, qa = sa * sa / dt, h = 0.5 * dt;
  const int s0 = sample_begin[f], s1 = sample_begin[f + 1];
  for (int s = s0; s < s1; ++s) {
    double w[3], a[3];
    for (int k = 0; k < 3; ++k) {
      w[k] = (gyro[3 * s + k] - bg[k]) * dt;
      a[k] = accel[3 * s + k] - ba[k];
    }
    double Ek[9], Jr[9], Ax[9], dRAx[9];
    exp_so3_jr(w, Ek, Jr);
    skew3(a, Ax);
    mul33(dR, Ax, dRAx);
    // P <- A P A^T + noise with A = [[E^T, 0, 0], [B, I, 0], [B dt/2, dt I, I]]
    // and B = -dR [a]x dt: first T = A P by block rows, then T A^T
    double Bm[9];
    for (int k = 0; k < 9; ++k) Bm[k] = -dRAx[k] * dt;
    double T00[9], T01[9], T02[9], BP0[9], BP1[9], BP2[9];
    mul33t(Ek, P00, T00);
    mul33t(Ek, P01, T01);
    mul33t(Ek, P02, T02);
    mul33(Bm, P00, BP0);
    mul33(Bm, P01, BP1);
    mul33(Bm, P02, BP2);
    double T10[9], T11[9], T12[9], T20[9], T21[9], T22[9];
    for (int x = 0; x < 3; ++x)
      for (int y = 0; y < 3; ++y) {
        const int k = 3 * x + y, kt = 3 * y + x;   // P_10 = P_01^T, P_20 = P_02^T, P_21 = P_12^T
        T10[k] = BP0[k] + P01[kt];
        T11[k] = BP1[k] + P11[k];
        T12[k] = BP2[k] + P12[k];
        T20[k] = h * BP0[k] + dt * P01[kt] + P02[kt];
        T21[k] = h * BP1[k] + dt * P11[k] + P12[kt];
        T22[k] = h * BP2[k] + dt * P12[k] + P22[k];
      }
    double TB0[9], TB1[9], TB2[9];
    mul33(T00, Ek, P00);
    mul3t3(T00, Bm, TB0);
    mul3t3(T10, Bm, TB1);
    mul3t3(T20, Bm, TB2);
    for (int k = 0; k < 9; ++k) {
      P01[k] = TB0[k] + T01[k];
      P02[k] = h * TB0[k] + dt * T01[k] + T02[k];
      P11[k] = TB1[k] + T11[k];
      P12[k] = h * TB1[k] + dt * T11[k] + T12[k];
      P22[k] = h * TB2[k] + dt * T21[k] + T22[k];
    }
    // gyroscope noise through J_r dt, accelerometer noise through dR dt and dR dt^2 / 2
    for (int x = 0; x < 3; ++x)
      for (int y = 0; y < 3; ++y) {
        double gg = 0.0, aa = 0.0;
        for (int k = 0; k < 3; ++k) {
          gg += Jr[3 * x + k] * Jr[3 * y + k];
          aa += dR[3 * x + k] * dR[3 * y + k];
        }
        P00[3 * x + y] += qg * dt * dt * gg;
        P11[3 * x + y] += qa * dt * dt * aa;
        P12[3 * x + y] += qa * 0.5 * dt * dt * dt * aa;
        P22[3 * x + y] += qa * 0.25 * dt * dt * dt * dt * aa;
      }
    // bias Jacobians (with dR, dv, J_Rg before this sample's update)
    double M1[9];
    mul33(dRAx, JRg, M1);
    for (int k = 0; k < 9; ++k) {
      Jpa[k] += Jva[k] * dt - 0.5 * dR[k] * dt * dt;
      Jpg[k] += Jvg[k] * dt - 0.5 * M1[k] * dt * dt;
      Jva[k] -= dR[k] * dt;
      Jvg[k] -= M1[k] * dt;
    }
    double EtJ[9];
    mul33t(Ek, JRg, EtJ);
    for (int k = 0; k < 9; ++k) JRg[k] = EtJ[k] - Jr[k] * dt;
    // the measurement
    double dRa[3];
    mv3(dR, a, dRa);
    for (int k = 0; k < 3; ++k) {
      dp[k] += dv[k] * dt + 0.5 * dRa[k] * dt * dt;
      dv[k] += dRa[k] * dt;
    }
    double nR[9];
    mul33(dR, Ek, nR);
    for (int k = 0; k < 9; ++k) dR[k] = nR[k];
  }
  const double dT = dt * (s1 - s0);
  for (int k = 0; k < 9; ++k) {
    pre[kPreDR + k] = dR[k];
    pre[kPreJRg + k] = JRg[k];
    pre[kPreJvg + k] = Jvg[k];
    pre[kPreJva + k] = Jva[k];
    pre[kPreJpg + k] = Jpg[k];
    pre[kPreJpa + k] = Jpa[k];
  }
  for (int k = 0; k < 3; ++k) {
    pre[kPreDv + k] = dv[k];
    pre[kPreDp + k] = dp[k];
    pre[kPreBa + k] = ba[k];
    pre[kPreBg + k] = bg[k];
  }
  pre[kPreDT] = dT;
  // information: the inverse of the 9x9 covariance (Cholesky), the bias
  // random walk 1 / (sigma^2 dT).  One sample's covariance has rank 6 (the
  // same accelerometer noise moves velocity and position), so an interval of
  // fewer than two samples gets NaN information.
  double* Info = pre + kPreInfo;
  for (int k = 0; k < 225; ++k) Info[k] = 0.0;
  double cov[81];
  for (int x = 0; x < 3; ++x)
    for (int y = 0; y < 3; ++y) {
      const int k = 3 * x + y, kt = 3 * y + x;
      cov[9 * x + y] = P00[k];
      cov[9 * x + 3 + y] = P01[k];
      cov[9 * x + 6 + y] = P02[k];
      cov[9 * (3 + x) + y] = P01[kt];
      cov[9 * (3 + x) + 3 + y] = P11[k];
      cov[9 * (3 + x) + 6 + y] = P12[k];
      cov[9 * (6 + x) + y] = P02[kt];
      cov[9 * (6 + x) + 3 + y] = P12[kt];
      cov[9 * (6 + x) + 6 + y] = P22[k];
    }
  const bool ok = s1 - s0 >= 2 && chol_n(cov, 9);
  for (int c = 0; c < 9; ++c) {
    double e[9] = {};
    e[c] = 1.0;
    if (ok) {
      lsolve(cov, 9, e);
      ltsolve(cov, 9, e);
    } else {
      for (int k = 0; k < 9; ++k) e[k] = __builtin_nan("");
    }
    for (int k = 0; k < 9; ++k) Info[15 * k + c] = e[k];
  }
  for (int k = 0; k < 3; ++k) {
    Info[15 * (9 + k) + 9 + k] = 1.0 / (sba * sba * dT);
    Info[15 * (12 + k) + 12 + k] = 1.0 / (sbg * sbg * dT);
  }
}

// ---------------------------------------------------------------------------
// IMU factors at the current state: one workgroup per factor
// ---------------------------------------------------------------------------

// Factor record in the workspace: H = J^T Lambda J (30 x 30), g = J^T Lambda r
// (30), r (15) and the factor's cost.
constexpr int kFH = 0, kFg = 900, kFr = 930, kFc = 945, kFRec = 946;
static_assert(kFRec <= kViFactorStride, "factor record stride");

// Lane 0's residual and Jacobian take most of it, from LDS, where all lanes put what it
// reads; four waves rather than one share the products: 14.5 us at nine factors with one
// wave, 10.6 with four, 9.5 with the staging.
constexpr int kFacThreads = 256;

__global__ __launch_bounds__(kFacThreads) void k_vi_fac(ViArgs V, int wbase) {
  __shared__ double sJ[450], sLJ[450], sI[225], sr[15];
  __shared__ double sX[24 + 18 + kPreInfo];   // both poses, both states, the factor's record up to Lambda
  const int wi = V.win_order[wbase + blockIdx.y];
  const WinDev W = V.win[wi];
  const int f = blockIdx.x, lane = threadIdx.x;
  if (f >= W.n_poses - 1) return;
  const int cur = V.state[wi].cur;
  const double* poses = (cur ? V.poses_b : V.poses) + 12 * W.pose_off;
  const double* states = (cur ? V.states_b : V.states) + 9 * W.pose_off;
  const double* pre = V.preint + (size_t)kPreStride * f;
  double* F = V.rec + (size_t)kViFactorStride * f;
  for (int e = lane; e < 450; e += kFacThreads) sJ[e] = 0.0;
  for (int e = lane; e < 225; e += kFacThreads) sI[e] = pre[kPreInfo + e];
  if (lane < 24 + 18 + kPreInfo)
    sX[lane] = lane < 24 ? poses[12 * f + lane] : lane < 42 ? states[9 * f + lane - 24] : pre[lane - 42];
  __syncthreads();
  if (lane == 0) {
    double r[15];
    imu_factor<true>(sX, sX + 24, sX + 12, sX + 33, sX + 42, V.g, r, sJ);
    for (int k = 0; k < 15; ++k) sr[k] = r[k];
  }
  __syncthreads();
  // Lambda J (15 x 30)
  for (int e = lane; e < 450; e += kFacThreads) {
    const int a = e / 30, c = e % 30;
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < 15; ++k) v += sI[15 * a + k] * sJ[30 * k + c];
    sLJ[e] = v;
  }
  __syncthreads();
  // H and g in one pass over the record's first 930 doubles
  for (int e = lane; e < 930; e += kFacThreads) {
    double v = 0.0;
    if (e < 900) {
      const int a = e / 30, c = e % 30;
#pragma unroll
      for (int k = 0; k < 15; ++k) v += sJ[30 * k + a] * sLJ[30 * k + c];
    } else {
      for (int k = 0; k < 15; ++k) v += sLJ[30 * k + e - 900] * sr[k];
    }
    F[e] = v;
  }
  if (lane < 15) F[kFr + lane] = sr[lane];
  if (lane == 0) F[kFc] = imu_cost1(sr, sI);
}

// ---------------------------------------------------------------------------
// elimination of the extra variables onto the poses: one workgroup per window
// ---------------------------------------------------------------------------

// H_xy of factor f staged as 12 x 18: rows (x_i, x_j) are H rows 0..5 and
// 15..20, columns (y_i, y_j) are H columns 6..14 and 21..29.
__device__ inline int hx_row(int q) { return q < 6 ? q : 9 + q; }
__device__ inline int hy_col(int c) { return c < 9 ? 6 + c : 12 + c; }

// t[i] -= b(r[i], M) m for all nine
template <int M>
__device__ __forceinline__ void sub_col(double (&t)[9], const double (&r)[9], double m) {
  __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 5, 10, 11) BA_FMAC_ROW(1, 6, 10, 11) BA_FMAC_ROW(2, 7, 10, 11)
                       BA_FMAC_ROW(3, 8, 10, 11) BA_FMAC_ROW(4, 9, 10, 11)
                   : "+&v"(t[0]), "+&v"(t[1]), "+&v"(t[2]), "+&v"(t[3]), "+&v"(t[4])
                   : "v"(r[0]), "v"(r[1]), "v"(r[2]), "v"(r[3]), "v"(r[4]), "v"(m), "n"(M));
  __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 4, 8, 9) BA_FMAC_ROW(1, 5, 8, 9) BA_FMAC_ROW(2, 6, 8, 9)
                       BA_FMAC_ROW(3, 7, 8, 9)
                   : "+&v"(t[5]), "+&v"(t[6]), "+&v"(t[7]), "+&v"(t[8])
                   : "v"(r[5]), "v"(r[6]), "v"(r[7]), "v"(r[8]), "v"(m), "n"(M));
}
// v -= b(s, M) u[M], M + 1 .. 8 in order
template <int M>
__device__ __forceinline__ void sub_chain(double& v, double s, const double (&u)[9]) {
  if constexpr (M < 8) {
    __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 1, 2, 4) BA_FMAC_ROW(0, 1, 3, 5)
                     : "+&v"(v)
                     : "v"(s), "v"(u[M]), "v"(u[M + 1]), "n"(M), "n"(M + 1));
    sub_chain<M + 2>(v, s, u);
  } else if constexpr (M == 8) {
    __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 1, 2, 3) : "+&v"(v) : "v"(s), "v"(u[8]), "n"(8));
  }
}
template <int I>
__device__ __forceinline__ void vi_back_steps(const double (&t)[9], const double (&r)[9], double (&u)[9]) {
  double v = t[I];
  sub_chain<I + 1>(v, r[I], u);
  u[I] = v * wave_bcast(r[I], I);
  if constexpr (I > 0) vi_back_steps<I - 1>(t, r, u);
}

// The elimination: one workgroup per window.  Its chain over the states (factor, then
// the forward and the backward substitution of all columns) is what it takes; the bytes
// are few.  Forward, each row of sixteen lanes holds two 9-wide panels in registers,
// w and p; its lanes 0-8 the rows of
//   w  A_k (damped, less C_k C_k^T): becomes L_k
//   p  A_{k,k+1}^T: becomes C_{k+1}
// and lanes 9-15 a column each of u_k - C_k w_{k-1}: becomes w_k.  The panels are
// factored column by column, right-looking, the pivot rows' entries broadcast within the
// sixteen lanes; as a column of C_{k+1} is done its products with C_{k+1}^T and w_k are
// added up for the next state.  No barrier, no LDS on the chain, and one pass for the
// factor, its panel and the substitution; an entry's updates keep their order, so the
// values are those of left-looking loops.  The panels are repeated for every seven
// lanes of columns.  The last waves add the pose-pose terms into the reduced system
// meanwhile.  Backward, a lane holds a column and reads L_k and C_{k+1} the same way.
// At 10 keyframes (9 free): 72 us with the factor on one thread and two barriers a state
// in each of three loops; 44 us with a wave's panel and the products' operands from LDS;
// 40 us with all operands by lane reads (issue: three instructions a product); 35 us so.
constexpr int kViLinThreads = 512;                     // threads of the elimination workgroup
constexpr int kViCols = 4 * 2 * (16 - 9);              // columns of a forward wave
constexpr int kViSweepWaves = 3;                       // forward waves; the others: pose-pose terms
constexpr int kViPoseThreads = kViLinThreads - 64 * kViSweepWaves;
// LDS doubles of the elimination beside X, for N states (the offsets in the kernel).
constexpr int vi_lin_doubles(int N) { return 81 * (4 * N - 1) + 216 * (N - 1) + 9 * N + 9; }
static_assert(kViSweepWaves * kViCols >= 6 * kViMaxStates + 1 && 64 * kViSweepWaves >= 6 * kViMaxStates + 1,
              "a lane per column");

template <bool XL>
__global__ __launch_bounds__(kViLinThreads) void k_vi_lin(ViArgs V, int wbase) {
  // the arrays of vi_lin_doubles(N), then X when both fit in LDS (XL)
  extern __shared__ __align__(16) double sDyn[];
  double* sM;
  if constexpr (XL) {
    sM = sDyn;
  } else {
    __shared__ double sStat[vi_lin_doubles(kViMaxStates)];
    sM = sStat;
  }
  __shared__ int sPose[kViMaxStates];   // pose of each free slot
  __shared__ int sOk;
  const int wi = V.win_order[wbase + blockIdx.x];
  const WinDev W = V.win[wi];
  const WinState& st = V.state[wi];
  const int tid = threadIdx.x;
  const int N = W.n_poses, nf = N - 1, nS = 6 * W.n_free, ncol = nS + 1;
  const double* F = V.rec;                           // per factor records
  // 9N x (nS + 1): A^-1 H_yx, then z = A^-1 g_y; row-major in LDS when it
  // fits (XL) and copied out at the end, since k_vi_cand reads it column by
  // column; otherwise column-major in the workspace throughout
  double* Xg = V.rec + (size_t)kViFactorStride * nf;
  double* X = XL ? sM + vi_lin_doubles(N) : Xg;
  const int xrow = XL ? ncol : 1, xcol = XL ? 1 : 9 * N;   // strides of X
  const int oO = 81 * N;               // after A_kk (damped): A_{k,k+1}
  const int oL = oO + 81 * (N - 1);    // L_k, the diagonal's reciprocals in its place
  const int oC = oL + 81 * N;          // C_{k+1} = A_{k+1,k} L_k^-T
  const int oH = oC + 81 * N;          // H_xy per factor
  const int oG = oH + 216 * (N - 1);   // g_y
  const int oZero = oG + 9 * N;        // nine zeros
  const int* fs = V.free_slot + W.pose_off;
  if (tid < N && fs[tid] >= 0) sPose[fs[tid]] = tid;
  if (tid == 0) sOk = 1;
  if (tid < 9) sM[oZero + tid] = 0.0;
  const int wave = tid >> 6, lane = tid & 63;
  // 1. stage A = H_yy + damping (block tridiagonal), A_{k,k+1}, H_xy and g_y:
  //    one index space over the four arrays, eight elements per thread and
  //    round, a round's reads (two per element, unconditional: an unused one
  //    reads F[0]) all in flight before its first LDS store
  const double lam = st.lambda;
  {
    const int nA = N * 81, nO = nf * 81, nH = nf * 216, nG = N * 9, ntot = nA + nO + nH + nG;
    constexpr int R = 8;
    for (int base = 0; base < ntot; base += R * blockDim.x) {
      long long i0[R], i1[R];
      double v0[R], v1[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = base + tid + r * (int)blockDim.x;
        i0[r] = -1;
        i1[r] = -1;
        if (e < nA) {
          const int k = e / 81, x = (e % 81) / 9, y = e % 9;
          if (k >= 1) i0[r] = (long long)kViFactorStride * (k - 1) + kFH + 30 * (21 + x) + 21 + y;
          if (k < nf) i1[r] = (long long)kViFactorStride * k + kFH + 30 * (6 + x) + 6 + y;
        } else if (e < nA + nO) {
          const int t = e - nA, f = t / 81, x = (t % 81) / 9, y = t % 9;
          i0[r] = (long long)kViFactorStride * f + kFH + 30 * (6 + x) + 21 + y;
        } else if (e < nA + nO + nH) {
          const int t = e - nA - nO, f = t / 216, q = (t % 216) / 18, c = t % 18;
          i0[r] = (long long)kViFactorStride * f + kFH + 30 * hx_row(q) + hy_col(c);
        } else if (e < ntot) {
          const int t = e - nA - nO - nH, k = t / 9, x = t % 9;
          if (k >= 1) i0[r] = (long long)kViFactorStride * (k - 1) + kFg + 21 + x;
          if (k < nf) i1[r] = (long long)kViFactorStride * k + kFg + 6 + x;
        }
        v0[r] = F[i0[r] >= 0 ? i0[r] : 0];
        v1[r] = F[i1[r] >= 0 ? i1[r] : 0];
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = base + tid + r * (int)blockDim.x;
        double v = 0.0;
        if (i0[r] >= 0) v += v0[r];
        if (i1[r] >= 0) v += v1[r];
        if (e < nA) {
          const int x = (e % 81) / 9, y = e % 9;
          if (x == y) v += lam * fmax(v, 1e-9);
          sM[e] = v;
        } else if (e < nA + nO) {
          sM[oO + e - nA] = v;
        } else if (e < ntot) {   // H_xy, g_y
          sM[oH + e - nA - nO] = v;
        }
      }
    }
  }
  __syncthreads();
  const int nblk = W.n_free * (W.n_free + 1) / 2;
  double* S = V.ssum + W.sum_off;
  double* sB = S + nblk * kBS;   // the reduced right-hand side (global)
  const int ptid = tid - 64 * kViSweepWaves;
  // 2. the last waves: the IMU cost at the current state (fixed order), for
  //    the first attempt, and the pose-pose terms
  if (ptid == 0) {
    double cf[kViMaxStates - 1];   // every factor's cost read before the sum
#pragma unroll
    for (int f = 0; f < kViMaxStates - 1; ++f) cf[f] = f < nf ? F[(size_t)kViFactorStride * f + kFc] : 0.0;
    double c = 0.0;
#pragma unroll
    for (int f = 0; f < kViMaxStates - 1; ++f)
      if (f < nf) c += cf[f];
    V.cost_a[wi] = c;
  }
  // pose-pose terms into the summed reduced system: upper entries of the
  // diagonal blocks, whole off-diagonal blocks (a, a + 1), -g into the rhs,
  // the diagonal into diag(U) (the damping uses the whole diagonal); every
  // read of a thread's elements goes out before its first update
  for (int base = 0; ptid >= 0 && base < N * 36; base += 2 * kViPoseThreads) {
    double fv[2][5], sv[2][4];
    long long so[2][4];
    int sa_[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int e = base + ptid + r * kViPoseThreads;
      const bool in = e < N * 36;
      const int a = in ? e / 36 : 0, rr = (e % 36) / 6, c = e % 6;
      const int sa = in ? fs[a] : -1;
      sa_[r] = sa;
      // F reads: diagonal-block terms of factors a - 1 and a, the off-diagonal
      // block of factor a, the rhs terms of factors a - 1 and a
      const long long fo[5] = {
          a >= 1 ? (long long)kViFactorStride * (a - 1) + kFH + 30 * (15 + rr) + 15 + c : 0,
          a < nf ? (long long)kViFactorStride * a + kFH + 30 * rr + c : 0,
          a < nf ? (long long)kViFactorStride * a + kFH + 30 * rr + 15 + c : 0,
          a >= 1 ? (long long)kViFactorStride * (a - 1) + kFg + 15 + rr : 0,
          a < nf ? (long long)kViFactorStride * a + kFg + rr : 0};
#pragma unroll
      for (int q = 0; q < 5; ++q) fv[r][q] = F[fo[q]];
      const int sb = (sa >= 0 && a < nf) ? fs[a + 1] : -1;
      so[r][0] = sa >= 0 && c >= rr ? (long long)kBS * blk_index(sa, sa, W.n_free) + 6 * rr + c : -1;
      so[r][1] = sa >= 0 && sb >= 0 ? (long long)kBS * blk_index(sa, sb, W.n_free) + 6 * rr + c : -1;
      so[r][2] = sa >= 0 && c == 0 ? (long long)(nblk * kBS + 6 * sa + rr) : -1;
      so[r][3] = sa >= 0 && c == rr ? (long long)(nblk * kBS + nS + 6 * sa + rr) : -1;
#pragma unroll
      for (int q = 0; q < 4; ++q) sv[r][q] = S[so[r][q] >= 0 ? so[r][q] : 0];
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int e = base + ptid + r * kViPoseThreads;
      const int sa = sa_[r];
      if (e >= N * 36 || sa < 0) continue;
      const int a = e / 36, rr = (e % 36) / 6, c = e % 6;
      double v = 0.0;
      if (a >= 1) v += fv[r][0];
      if (a < nf) v += fv[r][1];
      if (so[r][0] >= 0) S[so[r][0]] = sv[r][0] + v;
      if (so[r][3] >= 0) S[so[r][3]] = sv[r][3] + v;
      if (so[r][1] >= 0) S[so[r][1]] = sv[r][1] + fv[r][2];
      if (so[r][2] >= 0) {
        double gg = 0.0;
        if (a >= 1) gg += fv[r][3];
        if (a < nf) gg += fv[r][4];
        S[so[r][2]] = sv[r][2] - gg;
      }
    }
  }
  // 3. factor and forward sweep w_k = L_k^-1 (u_k - C_k w_{k-1}), state by state
  const int row = lane & 15;   // lane of its sixteen: panel rows 0-8, columns 9-15
  if (wave < kViSweepWaves && kViCols * wave < ncol) {
    // of the panels w and p: the lane's column, and where its entries of state k
    // stand: sM[q0 + step y] + sM[q1 + y]
    int col[2], lin[2], per[2], step[2], pa[2], h0[2], h1[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      col[q] = row < 9 ? ncol : kViCols * wave + 14 * (lane >> 4) + 7 * q + row - 9;
      lin[q] = oZero;
      per[q] = 0;
      step[q] = 1;
      pa[q] = -2;
      h0[q] = h1[q] = oZero;
      if (row < 9) {   // row of A_kk, row of A_{k,k+1}^T (past the last one: never used)
        lin[q] = q == 0 ? 9 * row : oO + row;
        per[q] = 81;
        step[q] = q == 0 ? 1 : 9;
      } else if (col[q] == nS) {
        lin[q] = oG;
        per[q] = 9;
      } else if (col[q] < nS) {
        // factor a - 1 holds pose a as x_j (rows 6 + r), factor a as x_i (rows r)
        pa[q] = sPose[col[q] / 6];
        const int r = col[q] % 6;
        if (pa[q] >= 1) h0[q] = oH + 216 * (pa[q] - 1) + 18 * (6 + r);
        if (pa[q] < nf) h1[q] = oH + 216 * pa[q] + 18 * r;
      }
    }
    auto entry = [&](int k, int q, double (&v)[9]) {
      int q0 = lin[q] + per[q] * k, q1 = oZero;
      const int d = k - pa[q];   // only next to the column's pose
      if (pa[q] >= 1 && (d == -1 || d == 0)) q0 = h0[q] + (d == 0 ? 9 : 0);
      if (pa[q] >= 0 && pa[q] < nf && (d == 0 || d == 1)) q1 = h1[q] + (d == 0 ? 0 : 9);
#pragma unroll
      for (int y = 0; y < 9; ++y) v[y] = sM[q0 + step[q] * y] + sM[q1 + y];
    };
    double w[9], p[9];
    entry(0, 0, w);
    entry(0, 1, p);
    double nw[9], np[9];
    entry(min(1, N - 1), 0, nw);
    entry(min(1, N - 1), 1, np);
    bool ok = true;
#pragma unroll 2
    for (int k = 0; k < N; ++k) {
      const int kn = min(k + 2, N - 1);
      double nw2[9], np2[9], aw[9], ap[9];   // the entries of the state after the next
      entry(kn, 0, nw2);
      entry(kn, 1, np2);
      // minus the sum for A_{k+1} (added to it whole), u_{k+1} less the products
#pragma unroll
      for (int y = 0; y < 9; ++y) {
        aw[y] = nw[y];
        ap[y] = row < 9 ? 0.0 : np[y];
      }
      ok = __builtin_amdgcn_readfirstlane(factor_panels<9>(w, p, aw, ap, row));   // the same in every lane and wave
      if (!ok) break;
      if (tid < 9) {
#pragma unroll
        for (int y = 0; y < 9; ++y) {
          sM[oL + 81 * k + 9 * tid + y] = w[y];
          sM[oC + 81 * k + 9 * tid + y] = p[y];
        }
      }
      double* o = X + (size_t)xrow * (9 * k);
      if (col[0] < ncol)
#pragma unroll
        for (int y = 0; y < 9; ++y) o[(size_t)xrow * y + (size_t)xcol * col[0]] = w[y];
      if (col[1] < ncol)
#pragma unroll
        for (int y = 0; y < 9; ++y) o[(size_t)xrow * y + (size_t)xcol * col[1]] = p[y];
#pragma unroll
      for (int y = 0; y < 9; ++y) {
        w[y] = row < 9 ? nw[y] + ap[y] : aw[y];
        p[y] = row < 9 ? np[y] : ap[y];
        nw[y] = nw2[y];
        np[y] = np2[y];
      }
    }
    if (!ok && tid == 0) sOk = 0;
  }
  __syncthreads();
  if (!sOk) {
    if (tid == 0) V.part_flag_a[W.chunk_begin] = 1;   // the reduce rejects the attempt
    return;
  }
  // 4. backward sweep u_k = L_k^-T (w_k - C_{k+1}^T u_{k+1}), a column per lane
  //    and, in lanes 0-8 of each sixteen, a row of C_{k+1} and of L_k
  if (64 * wave < ncol) {
    double* x = X + (size_t)xcol * min(tid, ncol - 1);
    const int lr = 9 * min(row, 8);
    double u[9], t[9], rc[9], rl[9];
#pragma unroll
    for (int y = 0; y < 9; ++y) {
      t[y] = x[(size_t)xrow * (9 * (N - 1) + y)];
      rl[y] = sM[oL + lr + 81 * (N - 1) + y];
      rc[y] = 0.0;
      u[y] = 0.0;
    }
#pragma unroll 2
    for (int k = N - 1; k >= 0; --k) {
      const int kn = max(k - 1, 0);
      double tn[9], rcn[9], rln[9];   // the next state's
#pragma unroll
      for (int y = 0; y < 9; ++y) {
        tn[y] = x[(size_t)xrow * (9 * kn + y)];
        rcn[y] = sM[oC + lr + 81 * kn + y];
        rln[y] = sM[oL + lr + 81 * kn + y];
      }
      {   // the last state has no C: its rc and u are zeros
        sub_col<0>(t, rc, u[0]);
        sub_col<1>(t, rc, u[1]);
        sub_col<2>(t, rc, u[2]);
        sub_col<3>(t, rc, u[3]);
        sub_col<4>(t, rc, u[4]);
        sub_col<5>(t, rc, u[5]);
        sub_col<6>(t, rc, u[6]);
        sub_col<7>(t, rc, u[7]);
        sub_col<8>(t, rc, u[8]);
      }
      vi_back_steps<8>(t, rl, u);
#pragma unroll
      for (int y = 0; y < 9; ++y) {
        if (tid < ncol) x[(size_t)xrow * (9 * k + y)] = u[y];
        t[y] = tn[y];
        rc[y] = rcn[y];
        rl[y] = rln[y];
      }
    }
  }
  __syncthreads();
  // 5. S <- S - H_xy X (upper blocks), rhs <- rhs + H_xy z; one row of a block
  //    (or of the rhs) per task
  // H(x_a row r, y_k) of the state k = a + J
  auto hrow = [&](int a, int r, auto J, double (&h)[9]) {
    const double* h0 = sM + (a >= 1 ? oH + 216 * (a - 1) + 18 * (6 + r) + (J < 0 ? 0 : 9) : oZero);
    const double* h1 = sM + (a < nf ? oH + 216 * a + 18 * r + (J > 0 ? 9 : 0) : oZero);
#pragma unroll
    for (int x = 0; x < 9; ++x) h[x] = J < 0 ? h0[x] : J > 0 ? h1[x] : h0[x] + h1[x];
  };
  const std::integral_constant<int, -1> kBefore;
  const std::integral_constant<int, 0> kAt;
  const std::integral_constant<int, 1> kAfter;
  // three rows of a block per thread: LDS reads bound it, and an entry of X is read
  // once for the three
  for (int e = tid; e < nblk * 2; e += kViLinThreads) {
    const int b = e / 2, r0 = 3 * (e % 2);
    int sa, sb;
    upper_pair(b, W.n_free, sa, sb);
    const int a = sPose[sa];
    double* so = S + kBS * b + 6 * r0;
    double acc[18], sv[18];
#pragma unroll
    for (int c = 0; c < 18; ++c) {
      acc[c] = 0.0;
      sv[c] = so[c];
    }
    auto add = [&](auto J) {
      double h[3][9];
#pragma unroll
      for (int r = 0; r < 3; ++r) hrow(a, r0 + r, J, h[r]);
      const double* xr = X + (size_t)xcol * (6 * sb) + (size_t)xrow * (9 * (a + J));
#pragma unroll
      for (int x = 0; x < 9; ++x)
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          const double v = xr[(size_t)xrow * x + (size_t)xcol * c];
#pragma unroll
          for (int r = 0; r < 3; ++r) acc[6 * r + c] += h[r][x] * v;
        }
    };
    if (a >= 1) add(kBefore);
    add(kAt);
    if (a < nf) add(kAfter);
#pragma unroll
    for (int c = 0; c < 18; ++c)
      if (sa != sb || c % 6 >= r0 + c / 6) so[c] = sv[c] - acc[c];
  }
  for (int e = kViLinThreads - 1 - tid; e < nS; e += kViLinThreads) {   // from the last wave on
    const int a = sPose[e / 6], r = e % 6;
    double v = 0.0;
    auto add = [&](auto J) {
      double h[9];
      hrow(a, r, J, h);
#pragma unroll
      for (int x = 0; x < 9; ++x) v += h[x] * X[(size_t)xcol * nS + (size_t)xrow * (9 * (a + J) + x)];
    };
    if (a >= 1) add(kBefore);
    add(kAt);
    if (a < nf) add(kAfter);
    sB[e] += v;
  }
  if (XL)
    for (int e = tid; e < 9 * N * ncol; e += kViLinThreads) Xg[e] = X[ncol * (e % (9 * N)) + e / (9 * N)];
}

// ---------------------------------------------------------------------------
// candidate velocities and biases, the IMU cost at the candidate
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_vi_cand(ViArgs V, int wbase) {
  const int wi = V.win_order[wbase + blockIdx.x];
  const WinDev W = V.win[wi];
  const WinState& st = V.state[wi];
  const int tid = threadIdx.x;
  if (st.fail) {
    if (tid == 0) V.cost_b[wi] = 0.0;
    return;
  }
  const int N = W.n_poses, nf = N - 1, nS = 6 * W.n_free, ncol = nS + 1;
  const int cur = st.cur;
  const double* states = (cur ? V.states_b : V.states) + 9 * W.pose_off;
  double* cstates = (cur ? V.states : V.states_b) + 9 * W.pose_off;
  const double* cposes = (cur ? V.poses : V.poses_b) + 12 * W.pose_off;
  const double* X = V.rec + (size_t)kViFactorStride * nf;
  const double* dx = V.dp + kDpStride * wi;
  // dy = -z - X dx
  for (int e = tid; e < 9 * N; e += blockDim.x) {
    const double* x = X + e;   // column-major: the lanes' reads are contiguous
    double v = -x[(size_t)9 * N * nS];
#pragma unroll 6
    for (int c = 0; c < nS; ++c) v -= x[(size_t)9 * N * c] * dx[c];
    cstates[e] = states[e] + v;
  }
  __syncthreads();
  __shared__ double sc[kViMaxStates];
  const double* pre = V.preint;
  for (int f = tid; f < nf; f += blockDim.x) {
    double r[15];
    imu_factor<false>(cposes + 12 * f, cstates + 9 * f, cposes + 12 * (f + 1), cstates + 9 * (f + 1),
                      pre + (size_t)kPreStride * f, V.g, r, nullptr);
    sc[f] = imu_cost1(r, pre + (size_t)kPreStride * f + kPreInfo);
  }
  __syncthreads();
  if (tid == 0) {
    double c = 0.0;
    for (int f = 0; f < nf; ++f) c += sc[f];
    V.cost_b[wi] = c;
  }
}

hipError_t launch_vi_preint(int n_factors, const int32_t* sample_begin, const double* gyro, const double* accel,
                            double dt, const double* bias_bar, const double* noise, double* out, hipStream_t st) {
  if (n_factors <= 0) return hipSuccess;
  // A workgroup per factor is five times as fast for a window's factors, but a CU holds
  // four of them and 256 factors of the other kernel: 100 us against 137 us for 2048
  // factors of 50 samples, 182 us against 139 us for 4096.
  constexpr int kPreMany = 2048;
  if (n_factors > kPreMany)
    hipLaunchKernelGGL(k_vi_preint_many, dim3((n_factors + 63) / 64), dim3(64), 0, st, n_factors, sample_begin,
                       gyro, accel, dt, bias_bar, noise[0], noise[1], noise[2], noise[3], out);
  else
    hipLaunchKernelGGL(k_vi_preint, dim3(n_factors), dim3(kPreThreads), 0, st, sample_begin, gyro, accel, dt,
                       bias_bar, noise[0], noise[1], noise[2], noise[3], out);
  return hipGetLastError();
}

void launch_vi_lin(const ViArgs& V, int wbase, int nwin, hipStream_t st) {
  if (nwin <= 0 || V.max_factors <= 0) return;
  hipLaunchKernelGGL(k_vi_fac, dim3(V.max_factors, nwin), dim3(kFacThreads), 0, st, V, wbase);
  // X (9N x (6 n_free + 1) doubles, n_free <= N) in LDS beside the other
  // arrays when the CU's 160 KB hold both (N <= 15; the limit is raised once
  // per process, as for the other kernels); otherwise, or if that fails, X
  // stays in the workspace.
  constexpr size_t kLds = 160 * 1024 - 1024;   // less the kernel's static LDS
  const int N = V.max_factors + 1;
  const size_t xb = sizeof(double) * (vi_lin_doubles(N) + 9 * (size_t)N * (6 * (size_t)N + 1));
  static std::once_flag once;
  static bool attr = false;
  std::call_once(once, [] {
    attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_vi_lin<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds) == hipSuccess;
  });
  if (attr && xb <= kLds)
    hipLaunchKernelGGL(k_vi_lin<true>, dim3(nwin), dim3(kViLinThreads), xb, st, V, wbase);
  else
    hipLaunchKernelGGL(k_vi_lin<false>, dim3(nwin), dim3(kViLinThreads), 0, st, V, wbase);
}

void launch_vi_cand(const ViArgs& V, int wbase, int nwin, hipStream_t st) {
  if (nwin > 0) hipLaunchKernelGGL(k_vi_cand, dim3(nwin), dim3(256), 0, st, V, wbase);
}

}  // namespace ba
