// gfx950 batched multi-view triangulation: every landmark re-estimated from its
// observations with the poses held fixed (paper Sec. 2.2, 3D module: new
// landmarks are triangulated from the multi-view observations of a keyframe
// before they enter the local map).
//
// One lane per landmark (a workgroup's landmarks ordered by observation count
// across its lanes); the landmark's observations are a contiguous range.  When
// the poses a workgroup reads span a range that, times the camera count, is at
// most 128, the world-to-camera transforms T_cb T_bw_i of that range are
// composed once into LDS, so each observation needs one transform and the
// Jacobian is A R_cw directly.  The workgroup's observations are then staged
// in LDS too (pixel minus principal point, transform, weight), read once in
// order: a lane walks its own range, so reading them from memory in every pass
// touched a cache line per lane and load, and those loads bound the kernel
// (1 M landmarks, 5.9 M observations, 12 passes: 607 -> 319 us).
//   start     the weighted least-squares intersection of the viewing rays,
//             (sum w (I - d d^T)) p0 = sum w (I - d d^T) c, by a 3x3 FP64
//             Cholesky; fewer than two views or a pivot <= 1e-10 trace marks
//             the landmark degenerate (NaN point, status 3); a start at depth
//             <= min_depth in any view is returned unrefined (status 4)
//   refine    exactly max_iters LM attempts on the robust reprojection cost:
//             V = sum w rho' J^T J, g = sum w rho' J^T r (J the 2x3 point
//             Jacobian A R_c R_i, accumulated in Real), (V + lambda
//             diag(max(V_kk, 1e-9))) d = -g by FP64 Cholesky, candidate p + d,
//             depth guard, accept iff the FP64 cost strictly drops
// Each candidate's pass also forms V, g there, so an accepted attempt needs no
// second pass.  Lanes share nothing: no barrier, no atomics.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "device.hpp"
#include "geometry.hpp"
#include "tri.hpp"

namespace ba {

constexpr int kTriPoseCache = 128;   // (pose, camera) transforms a workgroup keeps in LDS
// Stride of a transform's record in doubles: 16 are used, and 18 keep the records 16
// bytes aligned while records that lanes read together start in different banks.
constexpr int kTriRec = 18;
// Waves per SIMD the kernel is compiled for.  256 threads: four waves in FP32 measured
// 320 us against 350 with three, at 1 M landmarks; FP64 accumulators would spill there,
// so it keeps three.  Smaller workgroups, for longer tracks, are left at what they need
// (three).
template <typename Real, int NT>
constexpr int tri_waves() { return NT < 256 ? 2 : sizeof(Real) == 4 ? 4 : 3; }

// Cholesky solve of a 3x3 SPD system stored as (00, 01, 02, 11, 12, 22):
// x = A^-1 b.  False on a pivot <= floor or a non-finite one.
__device__ __forceinline__ bool solve3(const double* A, const double* b, double floor, double* x) {
  const double p0 = A[0];
  if (!(p0 > floor) || !isfinite(p0)) return false;
  const double i0 = rsqrt_nr(p0);
  const double l10 = A[1] * i0, l20 = A[2] * i0;
  const double p1 = A[3] - l10 * l10;
  if (!(p1 > floor) || !isfinite(p1)) return false;
  const double i1 = rsqrt_nr(p1);
  const double l21 = (A[4] - l20 * l10) * i1;
  const double p2 = A[5] - l20 * l20 - l21 * l21;
  if (!(p2 > floor) || !isfinite(p2)) return false;
  const double i2 = rsqrt_nr(p2);
  const double y0 = b[0] * i0;
  const double y1 = (b[1] - l10 * y0) * i1;
  const double y2 = (b[2] - l20 * y0 - l21 * y1) * i2;
  x[2] = y2 * i2;
  x[1] = (y1 - l21 * x[2]) * i1;
  x[0] = (y0 - l10 * x[1] - l20 * x[2]) * i0;
  return isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]);
}

// absent camera indices / weights read one constant entry (stride 0); global
// memory (not constant) keeps those loads global rather than flat
__device__ int kTriCamZero = 0;
__device__ double kTriWeightOne = 1.0;

// A workgroup's observations in LDS, from observation `first` on.
struct TriStage {
  long long first;
  const double2* d;     // u - cx, v - cy
  const double* w;      // weights (NULL: all 1)
  const uint8_t* rec;   // record of the composed transform
};

// The values are there before anything below uses them.
template <typename T, int N>
__device__ __forceinline__ void pin_all(T (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) __asm__ volatile("" : "+v"(v[k]));
}

// Ray start and LM refinement of landmark j (observations [o0, o1), indices
// already checked).  COMPOSED: P holds, per (pose i, camera c) at
// kTriRec ((i - pbase) n_cams + c), the camera record with the world-to-camera
// transform T_cb T_bw_i in place of T_cb (so the point goes to the camera in
// one transform and A R_cw is the Jacobian); otherwise P holds the poses
// (at 12 (i - pbase)) and the cameras come from sCam.  STAGED (composed): the
// observations come from G.  TIGHT (neither): the registers of four waves per SIMD.
// Left to the compiler they spilled 14, which the loop over the observations read back
// (200 poses in no order, 2.4 M landmarks of two views, 10 attempts: 732 us against 563
// of a kernel of three waves without staging; 537 us so).
template <typename Real, bool COMPOSED, bool STAGED, bool TIGHT = false>
__device__ __forceinline__ void tri_landmark(const TriArgs& A, int j, long long o0, long long o1,
                                             const double* sCam, const double* P, int pbase, const TriStage& G) {
  const DevSettings S = A.settings;
  const double kNaN = __builtin_nan("");
  const int* cp = A.obs_cam ? A.obs_cam : &kTriCamZero;
  const long long cstep = A.obs_cam ? 1 : 0;
  const double* wp = A.obs_w ? A.obs_w : &kTriWeightOne;
  const long long wstep = A.obs_w ? 1 : 0;
  auto finish = [&](int status, const double* p) {
    A.points[3 * (long long)j] = p ? p[0] : kNaN;
    A.points[3 * (long long)j + 1] = p ? p[1] : kNaN;
    A.points[3 * (long long)j + 2] = p ? p[2] : kNaN;
    if (A.reports) {
      ba_report r;
      r.initial_cost = kNaN;
      r.final_cost = kNaN;
      r.final_lambda = S.lambda_init;
      r.iters = 0;
      r.accepted = 0;
      r.chol_failures = 0;
      r.depth_rejects = 0;
      r.status = status;
      r.reserved = 0;
      A.reports[j] = r;
    }
  };
  if (o1 - o0 < 2) return finish(3, nullptr);

  // One observation: pose index (relative to pbase) and camera, or the transform's
  // record; pixel minus principal point; weight.  The loops below load observation
  // o + 1 while observation o is computed.
  struct Ob {
    int i, c;
    double u, v, w;
  };
  auto load = [&](long long o) {
    Ob b;
    if constexpr (STAGED) {
      const int k = (int)(o - G.first);
      const double2 d = G.d[k];
      b.u = d.x;
      b.v = d.y;
      b.i = G.rec[k];
      b.c = 0;
      b.w = G.w ? G.w[k] : 1.0;
    } else {
      b.i = A.obs_pose[o] - pbase;
      b.c = cp[o * cstep];
      b.u = A.obs_uv[2 * o];
      b.v = A.obs_uv[2 * o + 1];
      b.w = wp[o * wstep];
    }
    return b;
  };
  auto record = [&](const Ob& b) { return P + kTriRec * (STAGED ? b.i : b.i * A.n_cams + b.c); };

  // start: least-squares intersection of the viewing rays
  double M[6] = {0, 0, 0, 0, 0, 0}, mb[3] = {0, 0, 0};
  {
    Ob cur = load(o0);
    for (long long o = o0; o < o1; ++o) {
      const Ob nxt = load(o + 1 < o1 ? o + 1 : o);
      double Rcw[9], tcw[3];
      const double* C;
      if constexpr (COMPOSED) {
        C = record(cur);
#pragma unroll
        for (int k = 0; k < 9; ++k) Rcw[k] = C[4 + k];
#pragma unroll
        for (int a = 0; a < 3; ++a) tcw[a] = C[13 + a];
      } else {
        const double* T = P + 12 * cur.i;
        C = sCam + 16 * cur.c;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
          for (int b = 0; b < 3; ++b)
            Rcw[3 * a + b] = C[4 + 3 * a] * T[b] + C[5 + 3 * a] * T[4 + b] + C[6 + 3 * a] * T[8 + b];
          tcw[a] = C[4 + 3 * a] * T[3] + C[5 + 3 * a] * T[7] + C[6 + 3 * a] * T[11] + C[13 + a];
        }
      }
      const double v[3] = {(STAGED ? cur.u : cur.u - C[2]) / C[0], (STAGED ? cur.v : cur.v - C[3]) / C[1], 1.0};
      double d[3], ctr[3];
#pragma unroll
      for (int b = 0; b < 3; ++b) {   // world direction R_cw^T v and centre -R_cw^T t_cw
        d[b] = Rcw[b] * v[0] + Rcw[3 + b] * v[1] + Rcw[6 + b] * v[2];
        ctr[b] = -(Rcw[b] * tcw[0] + Rcw[3 + b] * tcw[1] + Rcw[6 + b] * tcw[2]);
      }
      const double in = rsqrt_nr(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
      d[0] *= in;
      d[1] *= in;
      d[2] *= in;
      const double dc = d[0] * ctr[0] + d[1] * ctr[1] + d[2] * ctr[2];
      const double w = cur.w;
      M[0] += w * (1.0 - d[0] * d[0]);
      M[1] -= w * d[0] * d[1];
      M[2] -= w * d[0] * d[2];
      M[3] += w * (1.0 - d[1] * d[1]);
      M[4] -= w * d[1] * d[2];
      M[5] += w * (1.0 - d[2] * d[2]);
#pragma unroll
      for (int a = 0; a < 3; ++a) mb[a] += w * (ctr[a] - d[a] * dc);
      cur = nxt;
    }
  }
  double p[3];
  if (!solve3(M, mb, 1e-10 * (M[0] + M[3] + M[5]), p)) return finish(3, nullptr);

  // one pass at point q: the robust cost, the number of depths <= min_depth,
  // and V (00 01 02 11 12 22), g
  auto pass = [&](const double* q, double& F, int& nbad, Real* V, Real* g) {
#pragma unroll
    for (int k = 0; k < 6; ++k) V[k] = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = 0;
    F = 0.0;
    nbad = 0;
    long long first = o0;
    // the first observation's addresses are formed anew in each pass
    if constexpr (TIGHT) __asm__ volatile("" : "+v"(first));
    Ob cur = load(first);
    for (long long o = o0; o < o1; ++o) {
      double T[COMPOSED ? 1 : 12];
      if constexpr (!COMPOSED) {
#pragma unroll
        for (int k = 0; k < 12; ++k) T[k] = P[12 * cur.i + k];
      }
      const Ob nxt = load(o + 1 < o1 ? o + 1 : o);
      if constexpr (TIGHT) pin_all(T);   // all reads go out first, none after a wait for another
      Real J0[3], J1[3];
      Lin<Real> L;
      if constexpr (COMPOSED) {
        // the record's transform takes the world point to the camera: the
        // rows of A R_cw are the Jacobian
        const double* C = record(cur);
        L = linearise<Real>(q, C, STAGED ? cur.u : cur.u - C[2], STAGED ? cur.v : cur.v - C[3], cur.w, S.huber_delta);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          J0[b] = L.a0[b];
          J1[b] = L.a1[b];
        }
      } else {
        const double* C = sCam + 16 * cur.c;
        double xb[3];
        Real R[9];   // R_i
#pragma unroll
        for (int a = 0; a < 3; ++a) xb[a] = T[4 * a] * q[0] + T[4 * a + 1] * q[1] + T[4 * a + 2] * q[2] + T[4 * a + 3];
#pragma unroll
        for (int k = 0; k < 9; ++k) R[k] = (Real)T[4 * (k / 3) + k % 3];
        if constexpr (TIGHT) pin_all(R);   // in FP32 over the linearisation: half the registers
        L = linearise<Real>(xb, C, cur.u - C[2], cur.v - C[3], cur.w, S.huber_delta);
        // J rows = (rows of A R_c) R_i
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          J0[b] = L.a0[0] * R[b] + L.a0[1] * R[3 + b] + L.a0[2] * R[6 + b];
          J1[b] = L.a1[0] * R[b] + L.a1[1] * R[3 + b] + L.a1[2] * R[6 + b];
        }
      }
      nbad += (L.Z > S.min_depth) ? 0 : 1;
      F += L.rho_w;
      const Real w1 = (Real)(L.wo * L.d1);
      int e = 0;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const Real wj0 = w1 * J0[r], wj1 = w1 * J1[r];
#pragma unroll
        for (int c = r; c < 3; ++c, ++e) V[e] = fma(wj1, J1[c], fma(wj0, J0[c], V[e]));
        g[r] = fma(wj1, L.r[1], fma(wj0, L.r[0], g[r]));
      }
      cur = nxt;
    }
    F *= 0.5;
  };

  Real V[6], g[3];
  double F;
  int nbad;
  pass(p, F, nbad, V, g);
  if (nbad > 0) return finish(4, p);
  const double F0 = F;
  double lam = S.lambda_init;
  int acc = 0, chol = 0, depth = 0;
  for (int it = 0; it < S.max_iters; ++it) {
    ba_iter_trace tr;
    tr.cost = F;
    tr.lambda = lam;
    tr.cand_cost = kNaN;
    tr.status = 0;
    double Ad[6] = {V[0], V[1], V[2], V[3], V[4], V[5]};
    const int dg[3] = {0, 3, 5};
#pragma unroll
    for (int k = 0; k < 3; ++k) Ad[dg[k]] += lam * fmax(Ad[dg[k]], 1e-9);
    const double mg[3] = {-(double)g[0], -(double)g[1], -(double)g[2]};
    double dlt[3];
    bool accept = false;
    if (!solve3(Ad, mg, 0.0, dlt)) {
      tr.status = 1;
      ++chol;
    } else {
      const double cand[3] = {p[0] + dlt[0], p[1] + dlt[1], p[2] + dlt[2]};
      Real Vc[6], gc[3];
      double Fc;
      int nb;
      pass(cand, Fc, nb, Vc, gc);
      if (nb > 0) {
        tr.status = 2;
        ++depth;
      } else {
        tr.cand_cost = Fc;
        accept = Fc < F;
      }
      if (accept) {
#pragma unroll
        for (int k = 0; k < 3; ++k) p[k] = cand[k];
#pragma unroll
        for (int k = 0; k < 6; ++k) V[k] = Vc[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) g[k] = gc[k];
        F = Fc;
        ++acc;
      }
    }
    lam = accept ? fmax(lam / S.lambda_down, S.lambda_min) : fmin(lam * S.lambda_up, S.lambda_max);
    tr.accepted = accept ? 1 : 0;
    if (A.traces) A.traces[(long long)j * S.max_iters + it] = tr;
  }
  A.points[3 * (long long)j] = p[0];
  A.points[3 * (long long)j + 1] = p[1];
  A.points[3 * (long long)j + 2] = p[2];
  if (A.reports) {
    ba_report r;
    r.initial_cost = F0;
    r.final_cost = F;
    r.final_lambda = lam;
    r.iters = S.max_iters;
    r.accepted = acc;
    r.chol_failures = chol;
    r.depth_rejects = depth;
    r.status = isfinite(F0) ? 0 : 1;
    r.reserved = 0;
    A.reports[j] = r;
  }
}

constexpr int kTriBins = 64;
// The kernel's static LDS: cameras, bins, order, ranges.
template <int NT>
constexpr int tri_static_lds() {
  return kMaxCams * 16 * 8 + 4 * (kTriBins + NT) + (NT / 64) * (3 * 4 + 2 * 8);
}

template <typename Real, int NT>
__global__ __launch_bounds__(NT, (tri_waves<Real, NT>())) void k_tri(TriArgs A, int pool) {
  constexpr int NW = NT / 64, kBins = kTriBins;
  __shared__ double sCam[kMaxCams * 16];
  extern __shared__ __align__(16) unsigned char sPool[];   // `pool` bytes: transforms, then the observations
  __shared__ int sBin[kBins];
  __shared__ int sOrder[NT];
  __shared__ int sRange[3][NW];
  __shared__ long long sObs[2][NW];
  const int tid = threadIdx.x;
  for (int k = tid; k < A.n_cams * 16; k += NT) sCam[k] = A.cams[k];
  // Lanes take the workgroup's landmarks in order of observation count, so that
  // the lanes of a wave run loops of similar length (a counting sort; the order of
  // equal counts is of no consequence, as a landmark's result depends on nothing
  // else).
  {
    const int jj = blockIdx.x * NT + tid;
    int n = kBins - 1;   // past the end: sorted last
    if (jj < A.n_points) {
      const long long m = (long long)A.point_obs_begin[jj + 1] - A.point_obs_begin[jj];
      n = m < 0 ? 0 : (m > kBins - 2 ? kBins - 2 : (int)m);
    }
    if (tid < kBins) sBin[tid] = 0;
    __syncthreads();
    atomicAdd(&sBin[n], 1);
    __syncthreads();
    if (tid < kBins) {   // exclusive prefix sum by the first wave
      const int own = sBin[tid];
      int v = own;
#pragma unroll
      for (int o = 1; o < kBins; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (tid >= o) v += u;
      }
      sBin[tid] = v - own;
    }
    __syncthreads();
    sOrder[atomicAdd(&sBin[n], 1)] = tid;
    __syncthreads();
  }
  const int j = blockIdx.x * NT + sOrder[tid];

  // the landmark's range, and the range of observations the workgroup reads
  int status = 0;
  long long o0 = 0, o1 = 0, omin = 1ll << 62, omax = -1;
  if (j < A.n_points) {
    o0 = A.point_obs_begin[j];
    o1 = A.point_obs_begin[j + 1];
    if (!(0 <= o0 && o0 <= o1 && o1 <= A.n_obs)) {
      status = 2;
      o0 = o1 = 0;
    } else if (o0 < o1) {
      omin = o0;
      omax = o1;
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const long long a = __shfl_xor(omin, m), b = __shfl_xor(omax, m);
    omin = a < omin ? a : omin;
    omax = b > omax ? b : omax;
  }
  if ((tid & 63) == 0) {
    sObs[0][tid >> 6] = omin;
    sObs[1][tid >> 6] = omax;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    omin = sObs[0][w] < omin ? sObs[0][w] : omin;
    omax = sObs[1][w] > omax ? sObs[1][w] : omax;
  }
  // Can the observations be staged, whatever the poses need?  (A landmark list in
  // no order, or a very long track, gives a range that does not fit.)
  const long long nobs = omax > omin ? omax - omin : 0;
  const int per = A.obs_w ? 25 : 17;   // bytes of one observation: two doubles, a byte [, the weight]
  const bool maybe = nobs > 0 && nobs * per + 32 <= pool;

  // structure checks and the range of pose indices: over the workgroup's
  // observations in order when they are to be staged (those of no valid index are
  // marked below), else over each landmark's own
  int pmin = 0x7fffffff, pmax = -1;
  bool bad = false;
  auto look = [&](long long o) {
    const int i = A.obs_pose[o], c = A.obs_cam ? A.obs_cam[o] : 0;
    const bool ok = i >= 0 && i < A.n_poses && c >= 0 && c < A.n_cams;
    if (ok) {
      pmin = i < pmin ? i : pmin;
      pmax = i > pmax ? i : pmax;
    }
    return ok;
  };
  if (maybe) {
    for (long long o = omin + tid; o < omax; o += NT) bad = !look(o) || bad;
  } else {
    for (long long o = o0; o < o1; ++o)
      if (!look(o)) status = 2;
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const int a = __shfl_xor(pmin, m), b = __shfl_xor(pmax, m);
    pmin = a < pmin ? a : pmin;
    pmax = b > pmax ? b : pmax;
  }
  bad = __any(bad);
  if ((tid & 63) == 0) {
    sRange[0][tid >> 6] = pmin;
    sRange[1][tid >> 6] = pmax;
    sRange[2][tid >> 6] = bad;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    pmin = sRange[0][w] < pmin ? sRange[0][w] : pmin;
    pmax = sRange[1][w] > pmax ? sRange[1][w] : pmax;
    bad = bad || sRange[2][w] != 0;
  }
  // only indices checked against n_poses count, so [pmin, pmax] is in range;
  // compose T_cb T_bw_i for every (pose, camera) the range holds
  const long long span = pmax >= pmin ? (long long)(pmax - pmin + 1) * A.n_cams : 0;
  const bool cached = span > 0 && span <= kTriPoseCache;
  double* sComp = reinterpret_cast<double*>(sPool);
  const int oD = cached ? (int)span * kTriRec * 8 : 0;   // bytes of the transforms, a multiple of 16
  static_assert(kTriPoseCache <= 255, "a staged observation's record is a byte, 255 marks a bad index");
  const bool staged = maybe && cached && oD + nobs * per <= pool;
  if (cached) {
    const int n = (int)span;
    for (int r = tid; r < n; r += NT) {
      const int i = pmin + r / A.n_cams, c = r % A.n_cams;
      const double* T = A.poses + 12 * (long long)i;
      const double* C = sCam + 16 * c;
      double* out = sComp + kTriRec * r;
      out[0] = C[0];
      out[1] = C[1];
      out[2] = C[2];
      out[3] = C[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
          out[4 + 3 * a + b] = C[4 + 3 * a] * T[b] + C[5 + 3 * a] * T[4 + b] + C[6 + 3 * a] * T[8 + b];
        out[13 + a] = C[4 + 3 * a] * T[3] + C[5 + 3 * a] * T[7] + C[6 + 3 * a] * T[11] + C[13 + a];
      }
    }
  }
  // the observations behind the transforms: pixels, weights, records
  TriStage G;
  double2* sD = reinterpret_cast<double2*>(sPool + oD);
  double* sW = reinterpret_cast<double*>(sPool + oD + 16 * (staged ? (int)nobs : 0));
  uint8_t* sRec = sPool + oD + (staged ? (int)nobs * (per - 1) : 0);
  if (staged) {
    for (int k = tid; k < (int)nobs; k += NT) {
      const long long o = omin + k;
      const int i = A.obs_pose[o], c = A.obs_cam ? A.obs_cam[o] : 0;
      const double u = A.obs_uv[2 * o], v = A.obs_uv[2 * o + 1];
      const bool ok = i >= 0 && i < A.n_poses && c >= 0 && c < A.n_cams;
      const double* C = sCam + 16 * (ok ? c : 0);
      sD[k] = make_double2(u - C[2], v - C[3]);
      if (A.obs_w) sW[k] = A.obs_w[o];
      sRec[k] = ok ? (uint8_t)((i - pmin) * A.n_cams + c) : 255;
    }
  }
  G.first = omin;
  G.d = sD;
  G.w = A.obs_w ? sW : nullptr;
  G.rec = sRec;
  __syncthreads();
  if (j >= A.n_points) return;
  if (staged) {
    for (long long o = o0; bad && o < o1; ++o)
      if (sRec[o - omin] == 255) status = 2;
  } else if (maybe && bad) {   // looked at in order above: this landmark's own still have to be
    for (long long o = o0; o < o1; ++o) {
      const int i = A.obs_pose[o], c = A.obs_cam ? A.obs_cam[o] : 0;
      if (i < 0 || i >= A.n_poses || c < 0 || c >= A.n_cams) status = 2;
    }
  }
  if (status) {
    const double kNaN = __builtin_nan("");
    A.points[3 * (long long)j] = kNaN;
    A.points[3 * (long long)j + 1] = kNaN;
    A.points[3 * (long long)j + 2] = kNaN;
    if (A.reports) {
      ba_report r;
      r.initial_cost = kNaN;
      r.final_cost = kNaN;
      r.final_lambda = A.settings.lambda_init;
      r.iters = 0;
      r.accepted = 0;
      r.chol_failures = 0;
      r.depth_rejects = 0;
      r.status = 2;
      r.reserved = 0;
      A.reports[j] = r;
    }
    return;
  }
  if (staged)
    tri_landmark<Real, true, true>(A, j, o0, o1, sCam, sComp, pmin, G);
  else if (cached)
    tri_landmark<Real, true, false>(A, j, o0, o1, sCam, sComp, pmin, G);
  else
    tri_landmark<Real, false, false, (NT == 256 && sizeof(Real) == 4)>(A, j, o0, o1, sCam, A.poses, 0, G);
}

template <typename Real, int NT>
static hipError_t launch_tri(const TriArgs& A, int pool) {
  const int blocks = (A.n_points + NT - 1) / NT;
  hipLaunchKernelGGL((k_tri<Real, NT>), dim3(blocks), dim3(NT), pool, (hipStream_t)A.stream, A, pool);
  return hipGetLastError();
}

// The pool of an NT-thread workgroup when `count` of them share a CU's LDS.
template <int NT>
constexpr int tri_pool(int count) {
  constexpr int kLds = 160 * 1024, kUnit = 1280;   // a CU's LDS, and the unit it is given out in
  return kLds / count / kUnit * kUnit - tri_static_lds<NT>() - 128;
}
static_assert(kTriPoseCache * kTriRec * 8 <= tri_pool<256>(4) && kTriPoseCache * kTriRec * 8 <= tri_pool<128>(6) &&
                  kTriPoseCache * kTriRec * 8 <= tri_pool<64>(6),
              "the transforms fit every pool");

// The largest count, max_count down to min_count, whose pool holds the observations of
// NT landmarks (by the mean per landmark, a sixteenth to spare) beside `poses`
// transforms; 0 when none does.
template <int NT>
static int tri_fit(double bytes, int poses, int max_count, int min_count) {
  for (int count = max_count; count >= min_count; --count)
    if (NT * bytes * 1.0625 + poses * (kTriRec * 8.0) <= tri_pool<NT>(count)) return count;
  return 0;
}

// Workgroup size and pool by the bytes of a landmark's observations: the kernel waits
// for memory and LDS most of the time, so what counts is how many landmarks a CU holds.
// 256 threads while three workgroups hold theirs (8 views without weights: a fixed 36 KB
// for 128 threads, three to a CU, took 359 us for 600 k landmarks, the unstaged kernel
// 357, this 246), 128 while four do (12 views: 345, 565, 304 us for 400 k), and 64 above,
// six to a CU while those fit and otherwise five (30 views: 600, 1040, 539 us for 160 k).
template <typename Real>
hipError_t run_triangulate(const TriArgs& A) {
  if (A.n_points <= 0) return hipSuccess;
  const double bytes = (double)A.n_obs / A.n_points * (A.obs_w ? 25 : 17);
  if (const int n = tri_fit<256>(bytes, 40, tri_waves<Real, 256>(), 3)) return launch_tri<Real, 256>(A, tri_pool<256>(n));
  if (const int n = tri_fit<128>(bytes, 40, 6, 4)) return launch_tri<Real, 128>(A, tri_pool<128>(n));
  return launch_tri<Real, 64>(A, tri_pool<64>(tri_fit<64>(bytes, 24, 6, 6) ? 6 : 5));
}

template hipError_t run_triangulate<float>(const TriArgs&);
template hipError_t run_triangulate<double>(const TriArgs&);

}  // namespace ba
