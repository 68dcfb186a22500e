// gfx950 kernels of the sliding-window sparse Levenberg-Marquardt bundle adjuster.
//
// The method (paper Sec. 2.2, Eq. 2 and Eq. 3, and the sentence after Eq. 3):
// per-observation pinhole reprojection residuals with a Huber kernel, the
// normal equations in blocks (U_i per pose, V_j per landmark, W_ij per
// pose-landmark pair), elimination of the landmarks by the Schur complement,
// a Cholesky solve of the reduced camera system for the poses, then point
// back-substitution.  One LM attempt is four launches over all windows of a
// batch:
//
//   pass_a     per chunk of landmarks: linearise every observation, reduce the
//              per-pair W, per-landmark V and per-pose U blocks, eliminate each
//              landmark (V* = L D L^T, Z = W L^-T |D|^-1/2) and accumulate the
//              chunk's private partial of S = U* - sum Z Z^T and of the reduced
//              right-hand side in LDS
//   sum        per window: the chunk partials added in FP64 in chunk order
//   reduce     per window: damp, blocked Cholesky (6x6 blocks) of S, two triangular solves,
//              candidate poses T' = Exp(dp) T
//   pass_b     per chunk: re-linearise (cheaper than storing W), back-substitute
//              dl_j, candidate points, robust cost of the candidate
//   accept     per window: compare costs, update lambda, switch state buffers;
//              done by every wave of the next pass_a for itself (the last one
//              by finalize), a launch only for windows of very many chunks
//              and in the per-stage timing solve
//
// The observation stream is coalesced SoA (du, dv, w) in landmark-major order.
// Within a workgroup, a tile of at most TP pairs is handled one thread per pair
// (linearisation, the pair's own Schur term, DPP sums per pose), one thread per
// landmark (3x3 elimination) and one thread per (off-diagonal target block,
// three rows) for the Schur products listed by the plan (no atomics).
// Every kernel of the adjoint (ADJ = true) reuses the same passes with the exact
// Hessian, lambda = 0 and the loss cotangent as right-hand side.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "device.hpp"
#include "vi.hpp"
#include "geometry.hpp"

namespace ba {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int xcd_chunk(int b, int G) {
  // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
  // contiguous run of chunks so that one window's chunks share an L2.
  const int q = G >> 3, r = G & 7;
  const int x = b & 7, k = b >> 3;
  return x * q + (x < r ? x : r) + k;
}


// Block accumulators of one pose-landmark pair.
template <typename Real>
struct PairAcc {
  Real U[21];   // upper triangle of the 6x6 pose block, row-major
  Real gp[6];   // pose gradient
  Real W[18];   // 6x3 pose-point block
  Real V[6];    // upper triangle of the 3x3 point block (00 01 02 11 12 22)
  Real gl[3];   // point gradient
};

template <typename Real>
__device__ __forceinline__ void pair_zero(PairAcc<Real>& A) {
#pragma unroll
  for (int k = 0; k < 21; ++k) A.U[k] = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) A.gp[k] = 0;
#pragma unroll
  for (int k = 0; k < 18; ++k) A.W[k] = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) A.V[k] = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) A.gl[k] = 0;
}

// Add one observation: the Gauss-Newton blocks with IRLS weight w rho', and in
// ADJ mode the remaining terms of the exact Hessian (second derivatives of the
// residual and the rho'' term).
template <typename Real, bool ADJ>
__device__ __forceinline__ void pair_add(PairAcc<Real>& A, const Lin<Real>& L, const Real* Rp,
                                         bool free_pose, const double* C) {
  Real Jp[2][6], Jl[2][3];
  const Real* ar[2] = {L.a0, L.a1};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const Real* a = ar[k];
    Jp[k][0] = a[0];
    Jp[k][1] = a[1];
    Jp[k][2] = a[2];
    Real c[3];
    cross3(L.xb, a, c);
    Jp[k][3] = c[0];
    Jp[k][4] = c[1];
    Jp[k][5] = c[2];
#pragma unroll
    for (int m = 0; m < 3; ++m) Jl[k][m] = Rp[m] * a[0] + Rp[3 + m] * a[1] + Rp[6 + m] * a[2];
  }
  const Real w1 = (Real)(L.wo * L.d1);
  Real wJp[2][6], wJl[2][3];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
#pragma unroll
    for (int m = 0; m < 6; ++m) wJp[k][m] = w1 * Jp[k][m];
#pragma unroll
    for (int m = 0; m < 3; ++m) wJl[k][m] = w1 * Jl[k][m];
  }
  if (free_pose) {
    int u = 0;
#pragma unroll
    for (int r = 0; r < 6; ++r) {
#pragma unroll
      for (int c = r; c < 6; ++c) A.U[u++] += wJp[0][r] * Jp[0][c] + wJp[1][r] * Jp[1][c];
      A.gp[r] += wJp[0][r] * L.r[0] + wJp[1][r] * L.r[1];
#pragma unroll
      for (int c = 0; c < 3; ++c) A.W[3 * r + c] += wJp[0][r] * Jl[0][c] + wJp[1][r] * Jl[1][c];
    }
  }
  {
    int v = 0;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
      for (int c = r; c < 3; ++c) A.V[v++] += wJl[0][r] * Jl[0][c] + wJl[1][r] * Jl[1][c];
      A.gl[r] += wJl[0][r] * L.r[0] + wJl[1][r] * L.r[1];
    }
  }
  if constexpr (ADJ) {
    // 2 w rho'' (J^T r)(J^T r)^T
    Real q[9];
#pragma unroll
    for (int m = 0; m < 6; ++m) q[m] = Jp[0][m] * L.r[0] + Jp[1][m] * L.r[1];
#pragma unroll
    for (int m = 0; m < 3; ++m) q[6 + m] = Jl[0][m] * L.r[0] + Jl[1][m] * L.r[1];
    const Real w2 = (Real)(2.0 * L.wo * L.d2);
    // w rho' sum_k r_k Hess(r_k) = w rho' (B^T Q B + M(a)),  B = [I, -[x_b]x, R_i]
    const double X = L.X, Y = L.Y;
    const double iz = recip_nr(L.Z);
    const Real pxz = (Real)(-(double)L.r[0] * C[0] * iz * iz);
    const Real pyz = (Real)(-(double)L.r[1] * C[1] * iz * iz);
    const Real pzz = (Real)(2.0 * ((double)L.r[0] * C[0] * X + (double)L.r[1] * C[1] * Y) * iz * iz * iz);
    Real c0[3], c1[3], c2[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      c0[m] = (Real)C[4 + m];
      c1[m] = (Real)C[7 + m];
      c2[m] = (Real)C[10 + m];
    }
    Real Q[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b)
        Q[a][b] = pxz * (c0[a] * c2[b] + c2[a] * c0[b]) + pyz * (c1[a] * c2[b] + c2[a] * c1[b]) +
                  pzz * c2[a] * c2[b];
    // columns of B
    Real Bc[9][3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      Real e[3] = {0, 0, 0};
      e[m] = 1;
      Bc[m][0] = e[0];
      Bc[m][1] = e[1];
      Bc[m][2] = e[2];
      cross3(e, L.xb, Bc[3 + m]);   // e_m x x_b = -[x_b]x e_m
      Bc[6 + m][0] = Rp[0 + m];
      Bc[6 + m][1] = Rp[3 + m];
      Bc[6 + m][2] = Rp[6 + m];
    }
    Real QB[9][3];
#pragma unroll
    for (int n = 0; n < 9; ++n)
#pragma unroll
      for (int a = 0; a < 3; ++a)
        QB[n][a] = Q[a][0] * Bc[n][0] + Q[a][1] * Bc[n][1] + Q[a][2] * Bc[n][2];
    Real ab[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) ab[m] = L.r[0] * L.a0[m] + L.r[1] * L.a1[m];
    const Real ax = ab[0] * L.xb[0] + ab[1] * L.xb[1] + ab[2] * L.xb[2];
    // M(a) entry (m, n) in (rho, phi, point) order
    auto Mab = [&](int m, int n) -> Real {
      if (m > n) {
        const int t = m;
        m = n;
        n = t;
      }
      if (m >= 3 && m < 6 && n >= 3 && n < 6) {
        const int a = m - 3, b = n - 3;
        return (Real)0.5 * (L.xb[a] * ab[b] + ab[a] * L.xb[b]) - (a == b ? ax : (Real)0);
      }
      if (m < 3 && n >= 3 && n < 6) {
        // M_rho,phi[a][b] = ([a]x)[a][b] / 2
        const int a = m, b = n - 3;
        Real sk;
        if (a == b) sk = 0;
        else if (a == 0) sk = (b == 1) ? -ab[2] : ab[1];
        else if (a == 1) sk = (b == 0) ? ab[2] : -ab[0];
        else sk = (b == 0) ? -ab[1] : ab[0];
        return (Real)0.5 * sk;
      }
      if (m >= 3 && m < 6 && n >= 6) {
        // M_phi,point = -[a]x R_i
        const int a = m - 3, c = n - 6;
        Real s[3];   // row a of [a]x
        if (a == 0) { s[0] = 0; s[1] = -ab[2]; s[2] = ab[1]; }
        else if (a == 1) { s[0] = ab[2]; s[1] = 0; s[2] = -ab[0]; }
        else { s[0] = -ab[1]; s[1] = ab[0]; s[2] = 0; }
        return -(s[0] * Rp[c] + s[1] * Rp[3 + c] + s[2] * Rp[6 + c]);
      }
      return (Real)0;
    };
    auto H2 = [&](int m, int n) -> Real {
      const Real t = Bc[m][0] * QB[n][0] + Bc[m][1] * QB[n][1] + Bc[m][2] * QB[n][2];
      return w1 * (t + Mab(m, n)) + w2 * q[m] * q[n];
    };
    if (free_pose) {
      int u = 0;
#pragma unroll
      for (int r = 0; r < 6; ++r) {
#pragma unroll
        for (int c = r; c < 6; ++c) A.U[u++] += H2(r, c);
#pragma unroll
        for (int c = 0; c < 3; ++c) A.W[3 * r + c] += H2(r, 6 + c);
      }
    }
    int v = 0;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = r; c < 3; ++c) A.V[v++] += H2(6 + r, 6 + c);
  }
}

// 3x3 symmetric L D L^T (no pivoting).  V = (v00 v01 v02 v11 v12 v22).
// ok = all pivots positive (spd) or merely non-zero (indef).
template <typename Real>
struct LDL3 {
  Real l10, l20, l21;
  Real isd[3];   // |d_k|^-1/2
  Real sg[3];    // sign(d_k)
};

// Reciprocal and reciprocal square root: the hardware approximations in FP32
// (about 1 ulp; the FP32 blocks carry far larger rounding already), IEEE in
// FP64, whose results are compared with the oracle at 1e-9.
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }
__device__ __forceinline__ float rsqrt_r(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt_r(double x) { return 1.0 / sqrt(x); }

template <typename Real>
__device__ __forceinline__ bool ldl3(const Real* V, bool spd, LDL3<Real>& F) {
  const Real d0 = V[0];
  const Real r0 = recip(d0);
  const Real l10 = V[1] * r0, l20 = V[2] * r0;
  const Real d1 = V[3] - l10 * l10 * d0;
  const Real l21 = (V[4] - l20 * l10 * d0) * recip(d1);
  const Real d2 = V[5] - l20 * l20 * d0 - l21 * l21 * d1;
  F.l10 = l10;
  F.l20 = l20;
  F.l21 = l21;
  const Real d[3] = {d0, d1, d2};
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const bool good = spd ? (d[k] > (Real)0) : (d[k] != (Real)0);
    ok = ok && good && isfinite((double)d[k]);
    const Real ad = fabs(d[k]);
    F.isd[k] = rsqrt_r(ad);
    F.sg[k] = d[k] < (Real)0 ? (Real)-1 : (Real)1;
  }
  return ok && isfinite((double)l10) && isfinite((double)l20) && isfinite((double)l21);
}

// solve L z = w (unit lower), then scale by |D|^-1/2: z_bar = |D|^-1/2 L^-1 w
template <typename Real>
__device__ __forceinline__ void ldl3_half(const LDL3<Real>& F, const Real* w, Real* z) {
  const Real z0 = w[0];
  const Real z1 = w[1] - F.l10 * z0;
  const Real z2 = w[2] - F.l20 * z0 - F.l21 * z1;
  z[0] = z0 * F.isd[0];
  z[1] = z1 * F.isd[1];
  z[2] = z2 * F.isd[2];
}

// x = V^-1 c = L^-T D^-1 L^-1 c
template <typename Real>
__device__ __forceinline__ void ldl3_solve(const LDL3<Real>& F, const Real* c, Real* x) {
  Real h[3];
  ldl3_half(F, c, h);
  const Real y0 = h[0] * F.isd[0] * F.sg[0];
  const Real y1 = h[1] * F.isd[1] * F.sg[1];
  const Real y2 = h[2] * F.isd[2] * F.sg[2];
  x[2] = y2;
  x[1] = y1 - F.l21 * x[2];
  x[0] = y0 - F.l10 * x[1] - F.l20 * x[2];
}

// V + lambda * diag(max(V_kk, 1e-9)) on the packed upper triangle
template <typename Real>
__device__ __forceinline__ void damp3(Real* V, double lam) {
  const int dI[3] = {0, 3, 5};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double v = (double)V[dI[k]];
    V[dI[k]] = (Real)(v + lam * (v > 1e-9 ? v : 1e-9));
  }
}

// Block-wide sum of a double, deterministic (fixed shuffle tree + fixed order).
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* scratch) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) scratch[wv] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int k = 0; k < NT / 64; ++k) t += scratch[k];
  __syncthreads();
  return t;   // valid in thread 0
}

// Sum of v and maximum of m over the workgroup (both valid in thread 0);
// scratch holds 2 NT / 64 doubles.
template <int NT>
__device__ __forceinline__ double block_sum_max(double v, double& m, double* scratch) {
  v = wave_sum(v);
  m = wave_max(m);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    scratch[wv] = v;
    scratch[NT / 64 + wv] = m;
  }
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0) {
    for (int k = 0; k < NT / 64; ++k) t += scratch[k];
    m = scratch[NT / 64];
    for (int k = 1; k < NT / 64; ++k) m = fmax(m, scratch[NT / 64 + k]);
  }
  __syncthreads();
  return t;
}

template <int NT>
__device__ __forceinline__ double block_max(double v, double* scratch) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) scratch[wv] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int k = 0; k < NT / 64; ++k) t = fmax(t, scratch[k]);
  __syncthreads();
  return t;   // valid in thread 0
}


// Per-chunk flags and costs of a window's chunks [c0, c1), reduced by one
// wave: lane l takes chunks c0 + l, c0 + l + 64, ... in order (four loads in
// flight), then a butterfly adds the lanes in a fixed order, so the sum is the
// same on every run.
__device__ __forceinline__ void wave_chunk_sums(const int32_t* flag, const double* cost, int c0, int c1,
                                                bool need_cost, int lane, int& f_out, double& F_out) {
  int f = 0;
  double F = 0.0;
  for (int c = c0 + lane; c < c1; c += 4 * 64) {
    int fl[4];
    double cs[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int cc = c + 64 * b;
      const bool in = cc < c1;
      fl[b] = in ? flag[cc] : 0;
      cs[b] = in && need_cost ? cost[cc] : 0.0;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      f |= fl[b];
      F += cs[b];
    }
  }
  f_out = __any(f);
  F_out = wave_bcast(wave_sum(F), 0);
}

// Accept or reject attempt it, by one wave: the chunks' candidate costs and depth
// flags summed, the costs compared, lambda and the current buffer updated.  `old`
// is the window's state after the attempt's reduction; every lane returns the
// state that the next attempt starts from, and the attempt's trace in tr.
template <typename Real>
__device__ __forceinline__ WinState decide(const WinState& old, const DevWork<Real>& K, const DevSettings& S, int wi,
                                           int n_free, int c0, int c1, int lane, ba_iter_trace& tr) {
  int depth = 0;
  double F = 0.0;   // (summed before anything of the state is looked at: one latency for both)
  wave_chunk_sums(K.part_flag_b, K.part_cost_b, c0, c1, true, lane, depth, F);
  WinState st = old;
  tr.cost = st.cost;
  tr.lambda = st.lambda;
  tr.cand_cost = __builtin_nan("");
  tr.accepted = 0;
  tr.status = 0;
  if (st.frozen) {   // frozen by an earlier attempt or by this one's gradient test
    tr.status = 3;
    return st;
  }
  // the step's max-norm for the step test: pose tangents and the chunks' point moves
  double sm = 0.0;
  if (S.step_tol > 0) {
    for (int e = lane; e < 6 * n_free; e += 64) sm = fmax(sm, fabs(K.dp[kDpStride * wi + e]));
    for (int c = c0 + lane; c < c1; c += 64) sm = fmax(sm, K.part_smax[c]);
    sm = wave_max(sm);
  }
  bool accept = false;
  if (st.fail) {
    tr.status = 1;
    st.chol_failures++;
  } else if (depth) {
    tr.status = 2;
    st.depth_rejects++;
  } else {
    F *= 0.5;
    if (K.vi_cost_b) F += K.vi_cost_b[wi];
    tr.cand_cost = F;
    st.cand_cost = F;
    accept = F < st.cost;
  }
  if (accept) {
    st.cost = tr.cand_cost;
    st.cur ^= 1;
    st.accepted++;
    st.lambda = fmax(st.lambda / S.lambda_down, S.lambda_min);
    if (S.step_tol > 0 && sm <= S.step_tol) st.frozen = 1;
  } else {
    st.lambda = fmin(st.lambda * S.lambda_up, S.lambda_max);
  }
  tr.accepted = accept ? 1 : 0;
  st.iters++;
  st.fail = 0;
  return st;
}

// The state that attempt it starts from is kept at parity it: the kernels of
// attempt it may then read the last one's while one wave writes the new one.
template <typename Real>
__device__ __forceinline__ WinState& state_at(const DevPlan& P, const DevWork<Real>& K, int it, int wi) {
  return K.state[(it & 1) * P.n_windows + wi];
}

// One wave decides attempt it - 1 and stores the state of attempt it and the trace.
template <typename Real>
__device__ __forceinline__ void put_decision(const DevPlan& P, const DevWork<Real>& K, const DevUser& U,
                                             const DevSettings& S, int it, int wi, int n_free, int c0, int c1,
                                             int lane) {
  ba_iter_trace tr;
  const WinState st = decide(state_at(P, K, it - 1, wi), K, S, wi, n_free, c0, c1, lane, tr);
  if (lane == 0) {
    state_at(P, K, it, wi) = st;
    if (U.traces) U.traces[(size_t)wi * S.max_iters + it - 1] = tr;
  }
}

// ---------------------------------------------------------------------------
// LDS layout of the chunk kernels
// ---------------------------------------------------------------------------

struct ChunkLds {
  // window caches
  static constexpr int kPose = 64 * 12;   // doubles
  static constexpr int kCam = 32 * 16;    // doubles
};

// Window caches of pass B: poses (current state) and camera table.
__device__ __forceinline__ void load_window(const DevPlan& P, const ChunkRec& W, const double* __restrict__ poses,
                                            double* sPose, double* sCam) {
  for (int k = threadIdx.x; k < W.n_poses * 12; k += blockDim.x) sPose[k] = poses[k];
  for (int k = threadIdx.x; k < W.n_cams * 16; k += blockDim.x) sCam[k] = P.cam[16 * W.cam_off + k];
}

// ---------------------------------------------------------------------------
// init, pack
// ---------------------------------------------------------------------------

template <typename Real>
__global__ void k_init(DevPlan P, DevWork<Real> K, DevSettings S) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= P.n_windows) return;
  WinState st;
  st.lambda = S.lambda_init;
  st.cost = 0.0;
  st.cand_cost = 0.0;
  st.init_cost = 0.0;
  st.cur = 0;
  st.fail = 0;
  st.accepted = st.chol_failures = st.depth_rejects = st.iters = st.status = st.frozen = 0;
  K.state[w] = st;
}

// Gather the user's observations (user order, FP64) into the plan-ordered SoA
// stream: du = u - cx, dv = v - cy (principal point removed before rounding to
// the stream precision), w.
template <typename Real>
__global__ void k_pack(DevPlan P, DevTiles T, DevWork<Real> K, DevUser U) {
  const int chunk = blockIdx.x;
  const int wi = T.chunk_window[chunk];
  const WinDev W = P.win[wi];
  const int t0 = T.chunk_tile_begin[chunk], t1 = T.chunk_tile_begin[chunk + 1];
  if (t1 <= t0) return;
  const int l0 = T.tile_lm_begin[t0], l1 = T.tile_lm_begin[t1];
  const int o0 = P.pair_obs_begin[P.lm_pair_begin[l0]];
  const int o1 = P.pair_obs_begin[P.lm_pair_begin[l1]];
  for (int o = o0 + threadIdx.x; o < o1; o += blockDim.x) {
    const int u = W.obs_off + P.obs_perm[o];
    const double* C = P.cam + 16 * (W.cam_off + P.obs_cam[o]);
    K.du[o] = (Real)(U.obs_uv[2 * u] - C[2]);
    K.dv[o] = (Real)(U.obs_uv[2 * u + 1] - C[3]);
    if (K.w) K.w[o] = (Real)U.obs_w[u];
  }
}

// ---------------------------------------------------------------------------
// pass A: linearise + per-landmark elimination + chunk partial of S
// ---------------------------------------------------------------------------

// One step of the segmented scan: v += (value of the source lane) where the
// source lane carries the same key.
template <typename Real, int N, int CTRL, int ROWMASK>
__device__ __forceinline__ void run_step(Real* v, int key) {
  const int k2 = dpp_i<CTRL, ROWMASK>(-2, key);
  const bool ok = k2 == key;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const Real t = dpp_r<CTRL, ROWMASK>(v[i]);
    if (ok) v[i] += t;
  }
}

// Inclusive prefix sums of v[0..N) over runs of lanes with equal key inside a
// wave (runs are contiguous: keys are sorted within the wave): after the call
// the last lane of each run holds the run's total.  DPP only (no LDS): four
// in-row shifts, then the two row broadcasts that carry a run across rows.
template <typename Real, int N>
__device__ __forceinline__ void run_sums(Real* v, int key) {
  run_step<Real, N, 0x111, 0xf>(v, key);   // row_shr:1
  run_step<Real, N, 0x112, 0xf>(v, key);   // row_shr:2
  run_step<Real, N, 0x114, 0xf>(v, key);   // row_shr:4
  run_step<Real, N, 0x118, 0xf>(v, key);   // row_shr:8
  run_step<Real, N, 0x142, 0xa>(v, key);   // row_bcast:15 into rows 1 and 3
  run_step<Real, N, 0x143, 0xc>(v, key);   // row_bcast:31 into rows 2 and 3
}

// Per-pose sums of pass A: U - Z sigma Z^T (21, upper), reduced rhs (6), diag(U) (6).
constexpr int kPoseSums = 33;

// Upper-triangle entry e (0..20) of a 6x6 block -> row-major offset r*6+c.
constexpr int kUpperOffC[21] = {0, 1, 2, 3, 4, 5, 7, 8, 9, 10, 11, 14, 15, 16, 17,
                                21, 22, 23, 28, 29, 35};

// The same offset for a run-time e (no table: an indexed table in constant
// memory would cost a memory access): row r has 6 - r entries.
__device__ __forceinline__ int upper_off(int e) {
  const int r = (e >= 6) + (e >= 11) + (e >= 15) + (e >= 18) + (e >= 20);
  const int start = 6 * r - r * (r - 1) / 2;
  return 7 * r + (e - start);
}

// Adds component k of a pose's run sum into the partial: U - Z sigma Z^T
// (upper triangle of the diagonal block), reduced rhs, diag(U) (LM only).
template <typename Real, bool ADJ>
__device__ __forceinline__ void pose_sum_add1(Real* sS, Real* sB, Real* sD, int nf, int s, int k,
                                              Real x) {
  if (k < 21) {
    sS[kBS * blk_index(s, s, nf) + upper_off(k)] += x;
  } else if (k < 27) {
    sB[6 * s + (k - 21)] += x;
  } else if (!ADJ) {
    sD[6 * s + (k - 27)] += x;
  }
}

template <typename Real, bool ADJ>
__device__ __forceinline__ void pose_sums_add(Real* sS, Real* sB, Real* sD, int nf, int s,
                                              const Real* v) {
  Real* D = sS + kBS * blk_index(s, s, nf);
#pragma unroll
  for (int k = 0; k < 21; ++k) D[kUpperOffC[k]] += v[k];
#pragma unroll
  for (int k = 0; k < 6; ++k) sB[6 * s + k] += v[21 + k];
  if (!ADJ) {
#pragma unroll
    for (int k = 0; k < 6; ++k) sD[6 * s + k] += v[27 + k];
  }
}

// Stored row stride of a pair's Z_bar (6 rows of 3), unpadded: the Schur units
// are bound by LDS bandwidth, and a padded row (4 floats) carries a quarter of
// dead bytes; the 18-word pair stride also spreads pairs over more banks.
template <typename Real>
struct ZRow {
  static constexpr int R = 3;
  static constexpr int S = 6 * R;
};

// Words of a tile's product list kept in registers between its load (tile
// start) and its store to LDS (after phase 2).
template <int TP>
struct ListRegs {
  static constexpr int N = TP >= 256 ? 12 : 4;
};

// LDS carve of pass A.  The camera table, the window's poses (FP64, staged
// once per work item: a tile's pairs read them right at its start) and the
// reduced-system partial are sized by the launch's largest window; the
// per-tile buffers by TP (a tile holds at most TP / 2 landmarks).  The pair ->
// landmark map is kept only for the adjoint's Schur units.
template <typename Real, int TP>
struct PassALds {
  static constexpr int NW = TP / 64;
  static size_t bytes(int np, int nc, int nf, int list_bytes, bool adj) {
    const size_t nblk = (size_t)nf * (nf + 1) / 2;
    return (size_t)(nc * 16 + np * 12 + 16) * sizeof(double) + ((adj ? TP : 0) + 4 + 8) * sizeof(int) +
           (nblk * kBS + 12 * (size_t)nf + (size_t)2 * NW * kPoseSums) * sizeof(Real) + 16 +
           ((size_t)TP * ZRow<Real>::S + (size_t)(TP / 2) * 12) * sizeof(Real) + 16 +
           ((size_t)list_bytes + 15) / 16 * 16;
  }
};

// Phase 4 of pass A for a tile of few target blocks: a unit owns CG entries of one
// row of a block and sums -Z_a[r] sigma Z_c^T over the block's products in list
// order (the same chain of FMAs per entry as the 2 x 6 units).  Two register sets
// in turn, so that a unit waits for LDS once per product; at its end the reads are
// clamped to the last product (read, not used).  LM only (sigma = 1).
template <typename Real, int CG>
__device__ __forceinline__ void schur_fine(const uint32_t* sLst, int nseg, const Real* sPZ, Real* sS) {
  constexpr int kZS = ZRow<Real>::S, ZR = ZRow<Real>::R;
  constexpr int NC = 6 / CG, UPS = 6 * NC;
  const uint16_t* sProd = reinterpret_cast<const uint16_t*>(sLst + nseg);
  const int u = threadIdx.x;   // one round: the caller checked nseg UPS <= threads
  if (u >= nseg * UPS) return;
  const uint32_t wd = sLst[u / UPS];
  const int row = (u % UPS) / NC, col = (u % NC) * CG;
  const int blk = wd & 1023, start = (wd >> 10) & 8191, len = wd >> 23;
  if (len == 0) return;
  Real acc[CG], a0[3], z0[CG][3], a1[3], z1[CG][3];
#pragma unroll
  for (int c = 0; c < CG; ++c) acc[c] = (Real)0;
  auto load = [&](uint32_t pp, Real (&a)[3], Real (&z)[CG][3]) {
    const Real* Za = sPZ + kZS * (pp & 255) + ZR * row;
    const Real* Zc = sPZ + kZS * (pp >> 8) + ZR * col;
#pragma unroll
    for (int m = 0; m < 3; ++m) a[m] = Za[m];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
      for (int m = 0; m < 3; ++m) z[c][m] = Zc[ZR * c + m];
  };
  auto madd = [&](const Real (&a)[3], const Real (&z)[CG][3]) {
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
      for (int m = 0; m < 3; ++m) acc[c] = fma(a[m], z[c][m], acc[c]);
  };
  const int end = start + len, last = end - 1;
  uint32_t i1 = sProd[min(start + 1, last)];
  load(sProd[start], a0, z0);
  for (int k = start;; k += 2) {
    const uint32_t i2 = sProd[min(k + 2, last)];
    load(i1, a1, z1);
    madd(a0, z0);
    if (k + 1 >= end) break;
    const uint32_t i3 = sProd[min(k + 3, last)];
    load(i2, a0, z0);
    madd(a1, z1);
    if (k + 2 >= end) break;
    i1 = i3;
  }
  Real* B = sS + kBS * blk + 6 * row + col;
#pragma unroll
  for (int c = 0; c < CG; ++c) B[c] -= acc[c];
}

// Threads of pass A, whatever the tile size: with 64-pair tiles (FP64 partials of
// more than 23 free poses take most of the LDS) one wave holds the pairs, and all
// four share the Schur units, which are most of such a tile's time.
constexpr int kPassAThreads = 256;

// FP32: at least two waves per SIMD (the register budget that LDS allows);
// FP64 runs one workgroup per CU anyway.
template <typename Real, int TP, bool ADJ>
__global__ __launch_bounds__(kPassAThreads, (sizeof(Real) == 4 ? 2 : 1)) void k_pass_a(DevPlan P, DevTiles T, DevWork<Real> K,
                                               DevUser U, DevSettings S, int it, int cls_begin,
                                               LdsDims D, int fused) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NT = kPassAThreads, NW = TP / 64;   // NW: waves that hold pairs
  constexpr int LR = ListRegs<TP>::N;
  constexpr int kZS = ZRow<Real>::S, ZR = ZRow<Real>::R;
  const ChunkRec W = T.chunk_rec[cls_begin + xcd_chunk(blockIdx.x, gridDim.x)];
  const int chunk = W.chunk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int4* trec = reinterpret_cast<const int4*>(T.tile_rec);
  const int4* prec = reinterpret_cast<const int4*>(T.pair_rec);
  // The global data of a tile is fetched one tile ahead, in three steps: tile
  // records two tiles ahead, pair records one tile ahead (both issued during
  // tile t - 1), and the pairs' points and first observations at the start of
  // tile t - 1 (their pair records are there by then).  The first tiles' records
  // come with the chunk's.
  const int t0 = W.t0, t1 = W.t1;
  int4 ta = W.ta0, tb = W.tb0, nta = W.ta1, ntb = W.tb1;
  int4 rec = make_int4(0, 0, 0, -1), nrec = rec;
  if (tid < ta.y) rec = prec[ta.x + tid];
  if (tid < nta.y) nrec = prec[nta.x + tid];
  // With `fused` no launch decided the last attempt: every wave does, from the same
  // sums in the same order (the loads above are in flight meanwhile).
  WinState st;
  if (!ADJ && fused && it > 0) {
    ba_iter_trace tr;
    st = decide(state_at(P, K, it - 1, W.wi), K, S, W.wi, W.n_free, W.chunk_begin, W.chunk_end, lane, tr);
  } else {
    st = state_at(P, K, it, W.wi);
  }
  if (!ADJ && st.frozen) return;   // the whole work item (every thread of it) returns
  const int cur = ADJ ? 0 : st.cur;
  const double lam = ADJ ? 0.0 : st.lambda;
  const double* poses = (cur ? K.poses_b : U.poses) + 12 * W.pose_off;
  const double* points = (cur ? K.points_b : U.points) + 3 * W.point_off;
  const int nf = W.n_free, nblk = nf * (nf + 1) / 2, nS = 6 * nf;

  double* sCam = reinterpret_cast<double*>(smem);             // nc * 16
  double* sPose = sCam + D.nc * 16;                           // np * 12
  double* sRed = sPose + D.np * 12;                           // 16
  int* sPL = reinterpret_cast<int*>(sRed + 16);               // TP (adjoint): pair -> tile-local landmark
  int* sFlag = sPL + (ADJ ? TP : 0);                          // 4
  int* sBndSlot = sFlag + 4;                                  // 8: slot of each edge run (or -1)
  Real* sS = reinterpret_cast<Real*>(sBndSlot + 8);           // nblk * kBS
  Real* sB = sS + nblk * kBS;                                 // nS
  Real* sD = sB + nS;                                         // nS
  Real* sBnd = sD + nS;                                       // 2 * NW * kPoseSums: edge-run sums
  // 16-byte aligned carve by offsets from the LDS base (integer casts of the
  // pointers would lose the LDS address space and turn every access into a
  // flat one)
  const int oPZ = ((int)(reinterpret_cast<unsigned char*>(sBnd + 2 * NW * kPoseSums) - smem) + 15) & ~15;
  Real* sPZ = reinterpret_cast<Real*>(smem + oPZ);           // TP * kZS
  Real* sPV = sPZ;                                            // TP * 9: V, g (phases 1-2, before Z)
  Real* sLF = sPZ + TP * kZS;                                 // TP / 2 * 12: landmark factors
  const int oLst = ((int)(reinterpret_cast<unsigned char*>(sLF + (TP / 2) * 12) - smem) + 15) & ~15;
  uint32_t* sLst = reinterpret_cast<uint32_t*>(smem + oLst);  // product lists (stored in phase 1)

  // a pair's point and first observation
  double px = 0, py = 0, pz = 0;
  Real du0 = 0, dv0 = 0, wo0 = 1;
  int cam0 = 0;
  // (threads without a pair read the window's first point and observation 0:
  // the loads are issued on every path, so the counter waits stay exact)
  auto fetch_pair = [&](const int4& r, bool on, double& x, double& y, double& z, Real& du, Real& dv, Real& wo,
                        int& cam) {
    const int o = on ? r.x : 0;
    const double* pt = points + 3 * (on ? r.y - W.point_off : 0);
    x = pt[0];
    y = pt[1];
    z = pt[2];
    cam = P.obs_cam[o];
    du = K.du[o];
    dv = K.dv[o];
    const Real wv = (K.w ? K.w : K.du)[o];   // a load on every path (the value is dropped without weights)
    wo = K.w ? wv : (Real)1;
  };
  if (t0 < t1) fetch_pair(rec, tid < ta.y, px, py, pz, du0, dv0, wo0, cam0);

  for (int k = tid; k < W.n_cams * 16; k += NT) sCam[k] = P.cam[16 * W.cam_off + k];
  for (int k = tid; k < W.n_poses * 12; k += NT) sPose[k] = poses[k];
  {
    // the partial starts 16 bytes aligned; the last store may run into sBnd,
    // which is written before it is read
    const int nz = (int)(((nblk * kBS + 2 * nS) * sizeof(Real) + 15) / 16);
    for (int k = tid; k < nz; k += NT) reinterpret_cast<float4*>(sS)[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (tid == 0) sFlag[0] = 0;
  __syncthreads();

  double cost = 0.0, gmax = 0.0;
  for (int t = t0; t < t1; ++t) {
    const int p0 = ta.x, nP = ta.y, l0 = ta.z, nL = ta.w;
    const int lw0 = tb.x, nseg = tb.y, nprod = tb.z;
    const int nwords = nseg + (nprod + 1) / 2;
    // this tile's pair: its pose (point and first observation are here
    // already), and the tile's list words
    const int q = (rec.z >> 8) & 255, pose = rec.z & 255, nobs = rec.z >> 16;
    const int slot = tid < nP ? rec.w : -1;
    const int o0 = rec.x, lm = rec.y;
    double Rt[12];
    if (tid < nP) {
      const double* pp = sPose + 12 * pose;
#pragma unroll
      for (int k = 0; k < 12; ++k) Rt[k] = pp[k];
    }
    // (unconditional, clamped to the tile's last landmark: loads issued on
    // every path keep the counter waits exact)
    const int lt = l0 + min(tid, nL > 0 ? nL - 1 : 0);
    const int lq0 = P.lm_pair_begin[lt] - p0, lq1 = P.lm_pair_begin[lt + 1] - p0;
    const bool lregs = nwords <= LR * NT;
    uint32_t lwv[LR];
    if (lregs) {
      // unconditional loads (clamped to the tile's last word; the table ends
      // with a padding word), so that waiting for them never waits for the
      // prefetches issued after them
      const int last = nwords > 0 ? nwords - 1 : 0;
#pragma unroll
      for (int k = 0; k < LR; ++k) lwv[k] = T.lists[lw0 + min(tid + k * NT, last)];
    }
    // In flight during this tile (issued after this tile's own loads: the
    // load counter retires in order, so waiting for the list words does not
    // wait for these): the tile record after the next one, and the next
    // tile's pairs' points and first observations.
    int4 nnta = nta, nntb = ntb;
    if (t + 2 < t1) {
      nnta = trec[2 * (t + 2)];
      nntb = trec[2 * (t + 2) + 1];
    }
    double npx = 0, npy = 0, npz = 0;
    Real ndu = 0, ndv = 0, nwo = 1;
    int ncam = 0;
    fetch_pair(nrec, t + 1 < t1 && tid < nta.y, npx, npy, npz, ndu, ndv, nwo, ncam);

    // ---- phase 1: thread t linearises its pair (free pairs sorted by slot)
    PairAcc<Real> A;
    pair_zero(A);
    if (tid < nP) {
      if (ADJ) sPL[q] = lm - l0;
      double xb[3];
#pragma unroll
      for (int a = 0; a < 3; ++a)
        xb[a] = Rt[4 * a] * px + Rt[4 * a + 1] * py + Rt[4 * a + 2] * pz + Rt[4 * a + 3];
      Real Rp[9];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) Rp[3 * a + b] = (Real)Rt[4 * a + b];
      {
        const double* C = sCam + 16 * cam0;
        const Lin<Real> L = linearise<Real>(xb, C, (double)du0, (double)dv0, (double)wo0, S.huber_delta);
        cost += L.rho_w;
        pair_add<Real, ADJ>(A, L, Rp, slot >= 0, C);
      }
      for (int o = o0 + 1; o < o0 + nobs; ++o) {
        const double* C = sCam + 16 * P.obs_cam[o];
        const double wo = K.w ? (double)K.w[o] : 1.0;
        const Lin<Real> L = linearise<Real>(xb, C, (double)K.du[o], (double)K.dv[o], wo,
                                            S.huber_delta);
        cost += L.rho_w;
        pair_add<Real, ADJ>(A, L, Rp, slot >= 0, C);
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) sPV[9 * q + k] = A.V[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) sPV[9 * q + 6 + k] = A.gl[k];
    }
    // this tile's product lists (the previous tile's phase 4 has ended)
    if (lregs) {
#pragma unroll
      for (int k = 0; k < LR; ++k) {
        const int i = tid + k * NT;
        if (i < nwords) sLst[i] = lwv[k];
      }
    } else {
      for (int i = tid; i < nwords; i += NT) sLst[i] = T.lists[lw0 + i];
    }
    __syncthreads();

    // ---- phase 2: one thread per landmark: V*, L D L^T, h
    if (tid < nL) {
      const int lmg = l0 + tid;
      Real V[6] = {0, 0, 0, 0, 0, 0}, g[3] = {0, 0, 0};
      // the landmark's pairs summed in order; the next pair's values are read
      // while the current ones are added (at the end the last pair is read
      // again, not used)
      if (lq0 < lq1) {
        Real x[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) x[k] = sPV[9 * lq0 + k];
        for (int qq = lq0; qq < lq1; ++qq) {
          const int nq = qq + 1 < lq1 ? qq + 1 : qq;
          Real y[9];
#pragma unroll
          for (int k = 0; k < 9; ++k) y[k] = sPV[9 * nq + k];
#pragma unroll
          for (int k = 0; k < 6; ++k) V[k] += x[k];
#pragma unroll
          for (int k = 0; k < 3; ++k) g[k] += x[6 + k];
#pragma unroll
          for (int k = 0; k < 9; ++k) x[k] = y[k];
        }
      }
      Real c[3];
      if (!ADJ) {
        gmax = fmax(gmax, fmax(fabs((double)g[0]), fmax(fabs((double)g[1]), fabs((double)g[2]))));
        damp3(V, lam);
        c[0] = -g[0];
        c[1] = -g[1];
        c[2] = -g[2];
      } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) c[k] = U.grad_points ? (Real)U.grad_points[3 * lmg + k] : (Real)0;
      }
      LDL3<Real> F;
      if (!ldl3(V, !ADJ, F)) sFlag[0] = 1;
      Real hb[3];
      ldl3_half(F, c, hb);
      Real* f = sLF + 12 * tid;
      f[0] = F.l10;
      f[1] = F.l20;
      f[2] = F.l21;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        f[3 + k] = F.isd[k];
        f[6 + k] = F.sg[k];
        f[9 + k] = hb[k];
      }
    }
    __syncthreads();
    // the pair records of the tile after the next one (its tile record has
    // arrived by now)
    // (unconditional, clamped: the values of threads without a pair are not used)
    const int4 nnrec = prec[nnta.x + min(tid, nnta.y > 0 ? nnta.y - 1 : 0)];

    // ---- phase 3: Z_bar = W L^-T |D|^-1/2 of this pair, its reduced rhs and
    // its own diagonal Schur term U - Z_bar sigma Z_bar^T (the products of a
    // pair with itself never enter the product lists), plus diag(U) for the
    // damping; then per-pose sums over adjacent lanes, added once per run
    Real v[kPoseSums];
    if (slot >= 0) {
      const Real* f = sLF + 12 * (lm - l0);
      LDL3<Real> F;
      F.l10 = f[0];
      F.l20 = f[1];
      F.l21 = f[2];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        F.isd[k] = f[3 + k];
        F.sg[k] = f[6 + k];
      }
      Real sh[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) sh[k] = f[6 + k] * f[9 + k];
      Real* Z = sPZ + kZS * q;
      Real z[6][3];
#pragma unroll
      for (int r = 0; r < 6; ++r) {
        ldl3_half(F, A.W + 3 * r, z[r]);
        Z[ZR * r] = z[r][0];
        Z[ZR * r + 1] = z[r][1];
        Z[ZR * r + 2] = z[r][2];
        if (ZR == 4) Z[ZR * r + 3] = (Real)0;
        v[21 + r] = (ADJ ? (Real)0 : -A.gp[r]) - (z[r][0] * sh[0] + z[r][1] * sh[1] + z[r][2] * sh[2]);
      }
      int e = 0;
#pragma unroll
      for (int r = 0; r < 6; ++r) {
        const Real zs0 = z[r][0] * F.sg[0], zs1 = z[r][1] * F.sg[1], zs2 = z[r][2] * F.sg[2];
        v[27 + r] = A.U[e];   // diagonal entry (r, r)
#pragma unroll
        for (int c = r; c < 6; ++c, ++e)
          v[e] = A.U[e] - (zs0 * z[c][0] + zs1 * z[c][1] + zs2 * z[c][2]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < kPoseSums; ++k) v[k] = (Real)0;
    }
    if (NW == NT / 64 || wave < NW) {
      run_sums<Real, kPoseSums>(v, slot);
      // The last lane of each run holds the run's sum.  A run inside the wave
      // is the only one of its pose in the tile (pairs are ordered by pose):
      // it adds into the partial directly.  The runs holding lane 0 or lane 63
      // may continue in the neighbouring waves: they go to this wave's two
      // edge slots, folded in phase 4.
      const int next = __shfl_down(slot, 1, 64);
      const int slot0 = __builtin_amdgcn_readlane(slot, 0);
      const int slot63 = __builtin_amdgcn_readlane(slot, 63);
      const bool tail = slot >= 0 && (lane == 63 || next != slot);
      if (lane == 0) {
        sBndSlot[2 * wave] = slot0 >= 0 ? slot0 : -1;
        sBndSlot[2 * wave + 1] = (slot63 >= 0 && slot63 != slot0) ? slot63 : -1;
      }
      if (tail) {
        if (slot == slot0 || lane == 63) {
          Real* dst = sBnd + (2 * wave + (slot == slot0 ? 0 : 1)) * kPoseSums;
#pragma unroll
          for (int k = 0; k < kPoseSums; ++k) dst[k] = v[k];
        } else {
          pose_sums_add<Real, ADJ>(sS, sB, sD, nf, slot, v);
        }
      }
    }
    __syncthreads();
    // edge runs of the waves, one thread per component (the targets are
    // diagonal blocks, rhs and diag(U); phase 4 below writes only
    // off-diagonal blocks).  The last wave does it: it gets the shortest Schur
    // units of every round.  A run spanning waves leaves its pieces in
    // consecutive edge slots: they are summed in wave order in registers and
    // added to the partial once.
    if (tid >= NT - kPoseSums) {
      const int k = tid - (NT - kPoseSums);
      int sl[2 * NW];
      Real x[2 * NW];
#pragma unroll
      for (int b = 0; b < 2 * NW; ++b) {
        sl[b] = sBndSlot[b];
        x[b] = sBnd[b * kPoseSums + k];
      }
      int cur = -1;
      Real acc = (Real)0;
#pragma unroll
      for (int b = 0; b < 2 * NW; ++b) {
        if (sl[b] < 0) continue;
        if (sl[b] == cur) {
          acc += x[b];
        } else {
          if (cur >= 0) pose_sum_add1<Real, ADJ>(sS, sB, sD, nf, cur, k, acc);
          cur = sl[b];
          acc = x[b];
        }
      }
      if (cur >= 0) pose_sum_add1<Real, ADJ>(sS, sB, sD, nf, cur, k, acc);
    }

    // ---- phase 4: Schur blocks.  Unit (segment, rows r0, r0 + 1) owns those rows
    // of one off-diagonal target block for this tile: it sums -Z_a[r] sigma Z_c^T
    // over the segment's products in registers and updates its rows of the partial
    // once.  A tile of few target blocks has long lists of products in each, which
    // one unit sums in series: as long as one round holds them, finer units shorten
    // that chain (a product of a one-entry unit is 6 LDS reads and 3 FMAs, of a
    // 2 x 6 unit 24 and 36; more LDS traffic in all, which bounds the phase once
    // the threads are busy: at 36 blocks 1 x 6 and 2 x 6 units measure alike).
    // FP64, 10 attempts, 2 x 6 units against these: 3 free poses 446 -> 409 us a
    // solve, 6 to 8 free poses 122 -> 117 us an attempt.  The adjoint has one
    // pass and keeps the coarse units.
    if (!ADJ && nseg * 36 <= NT) {
      schur_fine<Real, 1>(sLst, nseg, sPZ, sS);
    } else if (!ADJ && nseg * 12 <= NT) {
      schur_fine<Real, 3>(sLst, nseg, sPZ, sS);
    } else if (!ADJ && nseg * 6 <= NT) {
      schur_fine<Real, 6>(sLst, nseg, sPZ, sS);
    } else {
    const uint16_t* sProd = reinterpret_cast<const uint16_t*>(sLst + nseg);
      constexpr int RG = 2, UPS = 6 / RG;
      const int nun = nseg * UPS;
      for (int u = tid; u < nun; u += NT) {
        const uint32_t wd = sLst[u / UPS];
        const int r0 = (u % UPS) * RG;
        const int blk = wd & 1023, start = (wd >> 10) & 8191, len = wd >> 23;
        Real acc[RG][6];
#pragma unroll
        for (int i = 0; i < RG; ++i)
#pragma unroll
          for (int c = 0; c < 6; ++c) acc[i][c] = (Real)0;
        // Two register sets in turn: the Z rows of the next product (and the
        // index of the one after) are read while the current product is
        // multiplied, so a unit waits for LDS once per product.  At a unit's
        // end the reads are clamped to its last product (read, not used).
        Real a0[RG][3], z0[6][3], a1[RG][3], z1[6][3];
        auto load_rows = [&](uint32_t pp, Real (&a)[RG][3], Real (&z)[6][3]) {
          const int qa = pp & 255, qc = pp >> 8;
          const Real* Za = sPZ + kZS * qa + ZR * r0;
          const Real* Zc = sPZ + kZS * qc;
#pragma unroll
          for (int i = 0; i < RG; ++i)
#pragma unroll
            for (int m = 0; m < 3; ++m) a[i][m] = Za[ZR * i + m];
#pragma unroll
          for (int c = 0; c < 6; ++c)
#pragma unroll
            for (int m = 0; m < 3; ++m) z[c][m] = Zc[ZR * c + m];
          if (ADJ) {
            const Real* g = sLF + 12 * sPL[qa] + 6;
#pragma unroll
            for (int i = 0; i < RG; ++i)
#pragma unroll
              for (int m = 0; m < 3; ++m) a[i][m] *= g[m];
          }
        };
        // acc += a z^T as a chain of FMAs (one rounding per term)
        auto madd = [&](const Real (&a)[RG][3], const Real (&z)[6][3]) {
#pragma unroll
          for (int i = 0; i < RG; ++i)
#pragma unroll
            for (int c = 0; c < 6; ++c) {
              acc[i][c] = fma(a[i][0], z[c][0], acc[i][c]);
              acc[i][c] = fma(a[i][1], z[c][1], acc[i][c]);
              acc[i][c] = fma(a[i][2], z[c][2], acc[i][c]);
            }
        };
        const int end = start + len, last = end - 1;
        if (len > 0) {
          uint32_t i1 = sProd[min(start + 1, last)];
          load_rows(sProd[start], a0, z0);
          for (int k = start;; k += 2) {
            const uint32_t i2 = sProd[min(k + 2, last)];
            load_rows(i1, a1, z1);
            madd(a0, z0);
            if (k + 1 >= end) break;
            const uint32_t i3 = sProd[min(k + 3, last)];
            load_rows(i2, a0, z0);
            madd(a1, z1);
            if (k + 2 >= end) break;
            i1 = i3;
          }
        }
        Real* B = sS + kBS * blk + 6 * r0;
#pragma unroll
        for (int i = 0; i < RG; ++i)
#pragma unroll
          for (int c = 0; c < 6; ++c) B[6 * i + c] -= acc[i][c];
      }
    }
    __syncthreads();
    ta = nta;
    tb = ntb;
    nta = nnta;
    ntb = nntb;
    rec = nrec;
    nrec = nnrec;
    px = npx;
    py = npy;
    pz = npz;
    du0 = ndu;
    dv0 = ndv;
    wo0 = nwo;
    cam0 = ncam;
  }

  // ---- chunk partial out (the last tile's phase 4 ended with a barrier)
  Real* part = K.part + W.part_off;
#pragma unroll 4
  for (int k = tid; k < nblk * kBS + 2 * nS; k += NT) part[k] = sS[k];
  // the cost sum and the landmark-gradient maximum in one reduction
  double gm = gmax;
  const double tot = block_sum_max<NT>(cost, gm, sRed);
  if (tid == 0) {
    K.part_cost_a[chunk] = tot;
    K.part_flag_a[chunk] = sFlag[0];
    if (!ADJ) K.part_gmax[chunk] = gm;
  }
}

// ---------------------------------------------------------------------------
// reduce + blocked Cholesky of S + candidate poses (one workgroup per window)
// ---------------------------------------------------------------------------


// LDS stride of a 6x6 block in the reduction workgroup: dense, so every row
// pair of a block starts 16 bytes aligned and is read with one 128-bit LDS
// read (the chunk partials keep the odd stride kBS, which spreads the banks of
// the accumulating workgroups).
constexpr int kRS = 36;

// One item of the trailing update of step k of the blocked Cholesky in the
// reduction workgroup: rows 4 sub, 4 sub + 1 and 2 + sub (sub = 0, 1; a row pair is one
// 128-bit read) of one block of the upper pairs k + 2 <= i <= j (S_ij -= R_ki^T R_kj;
// block row k + 1 is the panel waves' own), n block rows, or, past their pairs, of the
// right-hand side (b_i -= R_ki^T y_k).  Every read is issued before the first product;
// each entry is summed over m in order and then subtracted.
__device__ __forceinline__ void trail_item(double* sS, double* sB, int k, int nf, int n, int e) {
  const int sub = e % 2, blkno = e / 2;
  const int rows[3] = {4 * sub, 4 * sub + 1, 2 + sub};
  const int npair = n * (n + 1) / 2;
  const bool rhs = blkno >= npair;
  int i, j = 0;
  if (rhs) i = blkno - npair;
  else upper_pair(blkno, n, i, j);
  const double* A = sS + kRS * blk_index(k, k + 2 + i, nf);
  double u[6][3];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    const double2 a01 = *reinterpret_cast<const double2*>(A + 6 * m + rows[0]);
    u[m][0] = a01.x;
    u[m][1] = a01.y;
    u[m][2] = A[6 * m + rows[2]];
  }
  if (!rhs) {
    const double* Bm = sS + kRS * blk_index(k, k + 2 + j, nf);
    double* D = sS + kRS * blk_index(k + 2 + i, k + 2 + j, nf);
    double v[6][6], d[3][6];
#pragma unroll
    for (int m = 0; m < 6; ++m)
#pragma unroll
      for (int c = 0; c < 6; c += 2) {
        const double2 b2 = *reinterpret_cast<const double2*>(Bm + 6 * m + c);
        v[m][c] = b2.x;
        v[m][c + 1] = b2.y;
      }
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 6; c += 2) {
        const double2 d2 = *reinterpret_cast<const double2*>(D + 6 * rows[r] + c);
        d[r][c] = d2.x;
        d[r][c + 1] = d2.y;
      }
    double acc[3][6];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 6; ++c) acc[r][c] = 0.0;
#pragma unroll
    for (int m = 0; m < 6; ++m)
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 6; ++c) acc[r][c] += u[m][r] * v[m][c];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 6; c += 2)
        *reinterpret_cast<double2*>(D + 6 * rows[r] + c) =
            make_double2(d[r][c] - acc[r][c], d[r][c + 1] - acc[r][c + 1]);
  } else {
    double yk[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) yk[m] = sB[6 * k + m];
    double* bi = sB + 6 * (k + 2 + i);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      double v = 0.0;
#pragma unroll
      for (int m = 0; m < 6; ++m) v += u[m][r] * yk[m];
      bi[rows[r]] -= v;
    }
  }
}

// Sum of a window's chunk partials in FP64 (grid: windows x slices).  The
// workgroup's 256 threads form G = W.sum_groups groups of 256 / G entry
// lanes; each thread keeps kSumE entries of its slice, group g adds chunks
// g, g + G, ... (four in flight per step) and the groups' sums are added in
// group order through LDS.  The partials of a window are contiguous, one
// per chunk, so the chunk addresses need no table lookup.
template <typename Real>
__global__ __launch_bounds__(256) void k_sum(DevPlan P, DevTiles T, DevWork<Real> K, DevUser U, DevSettings S, int it,
                                             int wbase, int fused) {
  __shared__ double sG[kSumE][256];
  const WinDev W = T.win_rec[wbase + blockIdx.x];
  // with `fused` the window's first workgroup also stores the decision on the last
  // attempt, which pass A has taken for itself
  const bool pending = fused && it > 0;
  const int frozen = state_at(P, K, pending ? it - 1 : it, W.self).frozen;
  if (pending && blockIdx.y == 0 && threadIdx.x >= 192)
    put_decision(P, K, U, S, it, W.self, W.n_free, W.chunk_begin, W.chunk_end, threadIdx.x & 63);
  if (frozen) return;
  const int nf = W.n_free, nblk = nf * (nf + 1) / 2;
  const int ne = nblk * kBS + 12 * nf;
  const int G = W.sum_groups, L = 256 / G;
  const int g = threadIdx.x / L, l = threadIdx.x - g * L;
  const int e0 = blockIdx.y * (L * kSumE);
  if (e0 >= ne) return;
  const int nch = W.chunk_end - W.chunk_begin;
  const Real* base = K.part + W.part_off;
  // loads are unconditional (entries past the end read the last entry and
  // are dropped), so a step's 16 loads are all in flight before the first
  // is waited for
  int ec[kSumE];
  bool in[kSumE];
#pragma unroll
  for (int k = 0; k < kSumE; ++k) {
    const int e = e0 + l + L * k;
    in[k] = e < ne;
    ec[k] = in[k] ? e : ne - 1;
  }
  double acc[kSumE];
#pragma unroll
  for (int k = 0; k < kSumE; ++k) acc[k] = 0.0;
  int c = g;
  for (; c + 3 * G < nch; c += 4 * G) {
    Real v[4][kSumE];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const Real* a = base + (int64_t)(c + j * G) * ne;
#pragma unroll
      for (int k = 0; k < kSumE; ++k) v[j][k] = a[ec[k]];
    }
#pragma unroll
    for (int k = 0; k < kSumE; ++k)
      acc[k] += (((double)v[0][k] + (double)v[1][k]) + (double)v[2][k]) + (double)v[3][k];
  }
  for (; c < nch; c += G) {
    const Real* a = base + (int64_t)c * ne;
#pragma unroll
    for (int k = 0; k < kSumE; ++k) acc[k] += (double)a[ec[k]];
  }
  double* dst = K.ssum + W.sum_off;
  if (G == 1) {
#pragma unroll
    for (int k = 0; k < kSumE; ++k)
      if (in[k]) dst[ec[k]] = acc[k];
    return;
  }
#pragma unroll
  for (int k = 0; k < kSumE; ++k) sG[k][threadIdx.x] = acc[k];
  __syncthreads();
  if (g == 0) {
#pragma unroll
    for (int k = 0; k < kSumE; ++k) {
      double t = sG[k][l];
      for (int h = 1; h < G; ++h) t += sG[k][h * L + l];
      if (in[k]) dst[ec[k]] = t;
    }
  }
}

template <typename Real, int NT, bool ADJ>
__global__ __launch_bounds__(NT) void k_reduce(DevPlan P, DevTiles T, DevWork<Real> K, DevUser U,
                                               DevSettings S, int it, int wbase) {
  extern __shared__ __align__(16) unsigned char smem[];
  const WinDev W = T.win_rec[wbase + blockIdx.x];
  const int wi = W.self;
  WinState& st = state_at(P, K, it, wi);
  const int tid = threadIdx.x;
  const int nf = W.n_free, nblk = nf * (nf + 1) / 2, nS = 6 * nf;
  double* sS = reinterpret_cast<double*>(smem);   // nblk * kRS
  double* sB = sS + nblk * kRS;                   // nS
  double* sD = sB + nS;                           // nS
  int* sFail = reinterpret_cast<int*>(sD + nS);   // 2 ints (one double): failure, freeze
  double* sMax = sD + nS + 1;                     // NT / 64 (<= 8): freeze test
  const int c0 = W.chunk_begin, c1 = W.chunk_end;
  const int ne = nblk * kBS + 2 * nS;
  if (!ADJ && st.frozen) return;
  {
    // the summed system, eight loads in flight per thread (up to 160 KB); the
    // blocks move from the summed partials' stride kBS to the dense kRS.  The
    // first round's loads go out before the chunk flags' chain of loads (wave 0).
    const double* src = K.ssum + W.sum_off;
    const int nb = nblk * kBS;
    constexpr int B = 8;
    int base = 0;
    do {   // once without free poses too (ne = 0): the flags are read in any case
      double v[B];
#pragma unroll
      for (int b = 0; b < B; ++b) v[b] = src[max(min(base + tid + b * NT, ne - 1), 0)];
      if (base == 0 && tid < 64) {
        const bool need_cost = !ADJ && it == 0;
        int f = 0;
        double F = 0.0;
        wave_chunk_sums(K.part_flag_a, K.part_cost_a, c0, c1, need_cost, tid, f, F);
        if (tid == 0) {
          sFail[0] = f;
          if (need_cost) {
            F *= 0.5;
            if (K.vi_cost_a) F += K.vi_cost_a[wi];
            st.cost = F;
            st.init_cost = F;
            if (!isfinite(F)) st.status = 1;
          }
        }
      }
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int e = base + tid + b * NT;
        if (e >= ne) continue;
        if (e < nb) {
          const int blk = e / kBS, r = e - kBS * blk;
          if (r < 36) sS[kRS * blk + r] = v[b];
        } else {
          sS[nblk * kRS + (e - nb)] = v[b];
        }
      }
      base += B * NT;
    } while (base < ne);
  }
  __syncthreads();
  if (!ADJ && S.grad_tol > 0) {
    // freeze test at this attempt's linearisation and damping: the reduced
    // right-hand side (summed) and the chunks' landmark gradient maxima; not
    // when a landmark block failed
    double m = 0.0;
    for (int e = tid; e < nS; e += NT) m = fmax(m, fabs(sB[e]));
    for (int c = c0 + tid; c < c1; c += NT) m = fmax(m, K.part_gmax[c]);
    const double gm = block_max<NT>(m, sMax);
    if (tid == 0) {
      sFail[1] = sFail[0] == 0 && gm <= S.grad_tol;
      if (sFail[1]) st.frozen = 1;
    }
    __syncthreads();
    if (sFail[1]) return;
  }
  const double lam = st.lambda;
  const double* poses = (ADJ || st.cur == 0 ? U.poses : K.poses_b) + 12 * W.pose_off;
  if (ADJ) {
    // right-hand side: tangent cotangent of the free poses plus the partials
    for (int i = tid; i < W.n_poses; i += NT) {
      const int f = P.free_slot[W.pose_off + i];
      if (f < 0) continue;
      const double* G = U.grad_poses + 12 * (W.pose_off + i);
      const double* Tp = poses + 12 * i;
      double M[9];
      for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
          M[3 * a + b] = G[4 * a] * Tp[4 * b] + G[4 * a + 1] * Tp[4 * b + 1] +
                         G[4 * a + 2] * Tp[4 * b + 2] + G[4 * a + 3] * Tp[4 * b + 3];
      sB[6 * f + 0] += G[3];
      sB[6 * f + 1] += G[7];
      sB[6 * f + 2] += G[11];
      sB[6 * f + 3] += M[7] - M[5];
      sB[6 * f + 4] += M[2] - M[6];
      sB[6 * f + 5] += M[3] - M[1];
    }
  } else {
    for (int e = tid; e < nS; e += NT) {
      const int f = e / 6, r = e % 6;
      const double d = sD[e];
      sS[kRS * blk_index(f, f, nf) + 7 * r] += lam * (d > 1e-9 ? d : 1e-9);
    }
  }
  // mirror the diagonal blocks (only their upper triangles were accumulated;
  // their diagonals, damped above, are not touched here)
  for (int e = tid; e < nf * 36; e += NT) {
    const int f = e / 36, r = (e % 36) / 6, c = e % 6;
    if (c < r) {
      double* D = sS + kRS * blk_index(f, f, nf);
      D[6 * r + c] = D[6 * c + r];
    }
  }
  // A landmark failure.  Read before the barrier: a pivot failure is raised in the same
  // word right behind it, and every wave has to go through the same barriers below.
  bool failed = sFail[0] != 0;
  __syncthreads();

  // Blocked Cholesky S = R^T R on 6x6 blocks (upper block storage), right-
  // looking.  The right-hand side rides along as one more column, so the
  // forward substitution R^T y = b happens inside the factorisation; the back
  // substitution runs in wave 0.  The chain over the block rows k bounds it.
  // The first waves keep the columns right of block column 0 and the right-hand
  // side, a column per lane throughout (kColWave a wave); lanes 0-5 of each row of
  // sixteen repeat the diagonal block (k, k), in w, and block (k, k + 1), in p.
  // Block row k is factored and solved in one pass over these panels, whose
  // products with block (k, k + 1) are the update of block row k + 1: added up in
  // registers along the way, they keep the other waves' update of the rows below
  // (with R_{k-1}, meanwhile) off the chain, and one barrier a block row is left (and
  // one after the panels' reads where two or three waves share them).
  // At 19 free poses: 47 us with a diagonal factor in one wave, a panel solve and
  // a trailing update a barrier apart each (3.8k cycles a block row); 40 us so.
  const int wave = tid >> 6, lane = tid & 63;
  if (!failed && nf > 0) {
    constexpr int kColWave = 80;
    const int nc = 6 * (nf - 1);                        // columns, then the right-hand side
    const int npw = nc / kColWave + 1;                  // panel waves (at most 3 of 8)
    const int row = lane & 15;
    const int oB = nblk * kRS;                          // sB behind sS
    // the lane's columns of w and p: block column j (kRhs: the right-hand side; 0: none), column c
    constexpr int kRhs = 1 << 20;
    int j[2], c[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int x = kColWave * wave + 20 * (lane >> 4) + 10 * q + row - 6;
      j[q] = row < 6 || x > nc ? 0 : x == nc ? kRhs : 1 + x / 6;
      c[q] = row < 6 ? row : x % 6;
    }
    double w[6], p[6], aw[6], ap[6], aq[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = aw[i] = ap[i] = aq[i] = 0.0;
    // Both sides go through the same barriers, so the branch has to be a scalar one; inside
    // one loop it cost 0.1 us a block row.
    if (__builtin_amdgcn_readfirstlane(wave < npw)) {
      for (int k = 0; k < nf; ++k) {
        const int dk = blk_index(k, k, nf);
        // where the panels' columns of block row k stand, and of R_{k-1,k+1}
        int o[2], s[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          s[q] = j[q] == kRhs ? 1 : 6;
          o[q] = j[q] == kRhs ? oB + 6 * k : kRS * (dk + (j[q] > k ? j[q] - k : 0)) + c[q];
        }
        if (row < 6) o[1] += k + 1 < nf ? kRS : 0;
        double sw[6], sp[6], qv[6];
        const double* Q = sS + kRS * (blk_index(k > 0 ? k - 1 : 0, k > 0 ? k : 0, nf) + (k > 0 && k + 1 < nf)) +
                          (row < 6 ? row : 0);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          qv[i] = Q[6 * i];
          sw[i] = sS[o[0] + s[0] * i];
          sp[i] = sS[o[1] + s[1] * i];
        }
        if (npw > 1) __syncthreads();   // another panel wave's stores below wait for these reads
        if (k > 0) {   // block (k, k + 1) less R_{k-1,k}^T R_{k-1,k+1}
#pragma unroll
          for (int i = 0; i < 6; ++i) aq[i] = 0.0;
#pragma unroll
          for (int m = 0; m < 6; ++m) sub_vec6(aq, p[m], qv[m]);
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          w[i] = sw[i] + (row < 6 ? ap[i] : aw[i]);
          p[i] = sp[i] + (row < 6 ? aq[i] : ap[i]);
          aw[i] = ap[i] = 0.0;
        }
        const bool ok = factor_panels<6>(w, p, aw, ap, row);
        if (tid == 0 && !ok) sFail[0] = 1;
        // the block's own columns once, its pivots' reciprocals on the diagonal
        if (j[0] > k || tid < 6) {
#pragma unroll
          for (int i = 0; i < 6; ++i) sS[o[0] + s[0] * i] = w[i];
        }
        if (j[1] > k) {
#pragma unroll
          for (int i = 0; i < 6; ++i) sS[o[1] + s[1] * i] = p[i];
        }
        __syncthreads();
      }
    } else {
      for (int k = 0; k < nf; ++k) {
        if (npw > 1) __syncthreads();
        const int n = k > 0 ? nf - k - 1 : 0;   // block rows below k, two items of three rows per block
        for (int e = tid - 64 * npw; e < n * (n + 3); e += NT - 64 * npw) trail_item(sS, sB, k - 1, nf, n, e);
        __syncthreads();
      }
    }
    failed = sFail[0] != 0;   // a failed pivot's NaNs have gone no further than S and b
  }
  // The candidate poses are wave 1's (a window has at most 64 poses): its reads
  // go out while wave 0 substitutes.
  int cslot = -1;
  double Tp[12];
  const bool cpose = !ADJ && wave == 1 && lane < W.n_poses;
  if (cpose) {
    cslot = P.free_slot[W.pose_off + lane];
#pragma unroll
    for (int k = 0; k < 12; ++k) Tp[k] = poses[12 * lane + k];
  }
  if (!failed && wave == 0 && nf > 0) {
    // back substitution R x = y in one wave.  Lane l keeps rows 3 l .. 3 l + 2
    // (all three in block row l / 2), so the rows of block k sit in lanes
    // 2 k and 2 k + 1 at register positions known at compile time; a lane's y is
    // not used any more once its block's x is known, so the lanes past it update
    // theirs with whatever they read.  Two register sets in turn: the next block's
    // reads are in flight while a block's chain runs.
    double y[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) y[t] = 3 * lane + t < nS ? sB[3 * lane + t] : 0.0;
    auto fetch = [&](int k, double (&dku)[15], double (&iv)[6], double (&bv)[18]) {
      const double* Dk = sS + kRS * blk_index(k, k, nf);
#pragma unroll
      for (int i = 0, q = 0; i < 6; ++i)
#pragma unroll
        for (int m = i + 1; m < 6; ++m, ++q) dku[q] = Dk[6 * i + m];
#pragma unroll
      for (int i = 0; i < 6; ++i) iv[i] = Dk[7 * i];
      const int l = lane < 2 * k ? lane : 0;   // lanes at or past block row k read block row 0
      const double* B = sS + kRS * blk_index(l >> 1, k, nf) + 18 * (l & 1);
#pragma unroll
      for (int m = 0; m < 18; m += 2) {
        const double2 b2 = *reinterpret_cast<const double2*>(B + m);
        bv[m] = b2.x;
        bv[m + 1] = b2.y;
      }
    };
    auto solve = [&](int k, const double (&dku)[15], const double (&iv)[6], const double (&bv)[18]) {
      double yv[6], x[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) yv[i] = wave_bcast(y[i % 3], 2 * k + i / 3);
#pragma unroll
      for (int i = 5; i >= 0; --i) {
        double v = yv[i];
        // dku holds row i's entries m = i + 1 .. 5 at q0(i) .. q0(i) + 4 - i
        const int q0 = 5 * i - i * (i - 1) / 2;
#pragma unroll
        for (int m = i + 1; m < 6; ++m) v -= dku[q0 + m - i - 1] * x[m];
        x[i] = v * iv[i];
      }
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 6; i += 2) *reinterpret_cast<double2*>(sB + 6 * k + i) = make_double2(x[i], x[i + 1]);
      }
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        double d = fma(bv[6 * t], x[0], bv[6 * t + 1] * x[1]);
#pragma unroll
        for (int i = 2; i < 6; ++i) d = fma(bv[6 * t + i], x[i], d);
        y[t] -= d;
      }
    };
    double d0[15], i0[6], b0[18], d1[15], i1[6], b1[18];
    fetch(nf - 1, d0, i0, b0);
    for (int k = nf - 1;; k -= 2) {
      fetch(k > 0 ? k - 1 : 0, d1, i1, b1);
      solve(k, d0, i0, b0);
      if (k == 0) break;
      fetch(k > 1 ? k - 2 : 0, d0, i0, b0);
      solve(k - 1, d1, i1, b1);
      if (k == 1) break;
    }
  }
  __syncthreads();
  double* dp = K.dp + kDpStride * wi;
  for (int e = tid; e < nS; e += NT) dp[e] = failed ? 0.0 : sB[e];
  if (ADJ) {
    if (tid == 0 && U.reports) U.reports[wi].chol_failures = failed ? 1 : 0;
    return;
  }
  if (tid == 0) st.fail = failed ? 1 : 0;
  if (failed) return;
  // candidate poses into the other buffer
  if (!cpose) return;
  double* Tc = (st.cur == 0 ? K.poses_b : U.poses) + 12 * (W.pose_off + lane);
  if (cslot < 0) {
#pragma unroll
    for (int k = 0; k < 12; ++k) Tc[k] = Tp[k];
    return;
  }
  double D[12];
  exp_se3(sB + 6 * cslot, D);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const double v = fma(D[4 * a + 2], Tp[8 + b], fma(D[4 * a], Tp[b], D[4 * a + 1] * Tp[4 + b]));
      Tc[4 * a + b] = b < 3 ? v : v + D[4 * a + 3];
    }
  }
}

// ---------------------------------------------------------------------------
// pass B: back-substitution + candidate cost (LM) / adjoint gather (ADJ)
// ---------------------------------------------------------------------------

template <typename Real, int TP, bool ADJ>
__global__ __launch_bounds__(TP) void k_pass_b(DevPlan P, DevTiles T, DevWork<Real> K, DevUser U,
                                               DevSettings S, int it, int cbase) {
  extern __shared__ __align__(16) unsigned char smem[];
  const ChunkRec W = T.chunk_rec[cbase + xcd_chunk(blockIdx.x, gridDim.x)];
  const int chunk = W.chunk, wi = W.wi;
  const int tid = threadIdx.x;
  const int4* trec = reinterpret_cast<const int4*>(T.tile_rec);
  const int4* prec = reinterpret_cast<const int4*>(T.pair_rec);
  const int t0 = W.t0, t1 = W.t1;
  int4 ta = W.ta0;
  int4 rec = make_int4(0, 0, 0, -1);
  if (tid < ta.y) rec = prec[ta.x + tid];
  const WinState& st = state_at(P, K, it, wi);
  if (!ADJ && (st.fail || st.frozen)) {
    if (tid == 0) {
      K.part_cost_b[chunk] = 0.0;
      K.part_flag_b[chunk] = 0;
      K.part_smax[chunk] = 0.0;
    }
    return;
  }
  const int cur = ADJ ? 0 : st.cur;
  const double lam = ADJ ? 0.0 : st.lambda;
  const double* poses = (cur ? K.poses_b : U.poses) + 12 * W.pose_off;
  const double* points = (cur ? K.points_b : U.points) + 3 * W.point_off;
  const double* cposes = (cur ? U.poses : K.poses_b) + 12 * W.pose_off;
  double* cpoints = (cur ? U.points : K.points_b) + 3 * W.point_off;
  const int nS = 6 * W.n_free;

  double* sPose = reinterpret_cast<double*>(smem);
  double* sCam = sPose + ChunkLds::kPose;
  double* sPoseC = sCam + ChunkLds::kCam;          // 64 * 12 (candidate poses)
  double* sDp = sPoseC + ChunkLds::kPose;          // kDpStride
  double* sLP = sDp + kDpStride;                   // TP * 3 (candidate point / a_l)
  double* sRed = sLP + 3 * TP;                     // 16
  int* sFlag = reinterpret_cast<int*>(sRed + 16);  // 4
  Real* sPV = reinterpret_cast<Real*>(sFlag + 4);  // TP * 12: V, g, W^T dp per pair

  // A tile's global data is fetched during the tile before it: each pair's
  // point and first observation (after the pair records arrive, behind phase
  // 3), each landmark's pair range and point (behind the whole tile).
  double px = 0, py = 0, pz = 0;
  Real du0 = 0, dv0 = 0, wo0 = 1;
  int cam0 = 0;
  auto fetch_pair = [&](const int4& r, double& x, double& y, double& z, Real& du, Real& dv, Real& wo,
                        int& cam) {
    const double* pt = points + 3 * (r.y - W.point_off);
    x = pt[0];
    y = pt[1];
    z = pt[2];
    cam = P.obs_cam[r.x];
    du = K.du[r.x];
    dv = K.dv[r.x];
    wo = K.w ? K.w[r.x] : (Real)1;
  };
  int lb0 = 0, lb1 = 0;
  double lx = 0, ly = 0, lz = 0;
  auto fetch_lm = [&](int lmt, int& b0, int& b1, double& x, double& y, double& z) {
    b0 = P.lm_pair_begin[lmt];
    b1 = P.lm_pair_begin[lmt + 1];
    const double* pt = points + 3 * (lmt - W.point_off);
    x = pt[0];
    y = pt[1];
    z = pt[2];
  };
  if (t0 < t1) {
    if (tid < ta.y) fetch_pair(rec, px, py, pz, du0, dv0, wo0, cam0);
    if (tid < ta.w) fetch_lm(ta.z + tid, lb0, lb1, lx, ly, lz);
  }
  load_window(P, W, poses, sPose, sCam);
  if (!ADJ)
    for (int k = tid; k < W.n_poses * 12; k += TP) sPoseC[k] = cposes[k];
  for (int k = tid; k < nS; k += TP) sDp[k] = K.dp[kDpStride * wi + k];
  if (tid == 0) sFlag[0] = 0;
  __syncthreads();

  double cost = 0.0, smax = 0.0;
  for (int t = t0; t < t1; ++t) {
    // the tile's pairs in the plan's thread order; q is the pair's index in
    // landmark order (the layout of the per-pair LDS rows)
    const int p0 = ta.x, nP = ta.y, l0 = ta.z, nL = ta.w;
    const int q = (rec.z >> 8) & 255, pose = rec.z & 255, nobs = rec.z >> 16;
    const int slot = rec.w, o0 = rec.x, lm = rec.y;
    const int j = lm - l0;
    int4 nta = ta;
    if (t + 1 < t1) nta = trec[2 * (t + 1)];
    // the next tile's landmarks (their tile record is needed first)
    int nlb0 = 0, nlb1 = 0;
    double nlx = 0, nly = 0, nlz = 0;
    if (t + 1 < t1 && tid < nta.w) fetch_lm(nta.z + tid, nlb0, nlb1, nlx, nly, nlz);

    // ---- phase 1: per pair: W, V, g at the current state and W^T dp
    if (tid < nP) {
      const double* Rt = sPose + 12 * pose;
      double xb[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) xb[a] = Rt[4 * a] * px + Rt[4 * a + 1] * py + Rt[4 * a + 2] * pz + Rt[4 * a + 3];
      Real Rp[9];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) Rp[3 * a + b] = (Real)Rt[4 * a + b];
      PairAcc<Real> A;
      pair_zero(A);
      {
        const double* C = sCam + 16 * cam0;
        const Lin<Real> L = linearise<Real>(xb, C, (double)du0, (double)dv0, (double)wo0, S.huber_delta);
        pair_add<Real, ADJ>(A, L, Rp, slot >= 0, C);
      }
      for (int o = o0 + 1; o < o0 + nobs; ++o) {
        const double* C = sCam + 16 * P.obs_cam[o];
        const double wo = K.w ? (double)K.w[o] : 1.0;
        const Lin<Real> L = linearise<Real>(xb, C, (double)K.du[o], (double)K.dv[o], wo,
                                            S.huber_delta);
        pair_add<Real, ADJ>(A, L, Rp, slot >= 0, C);
      }
      Real wtd[3] = {0, 0, 0};
      if (slot >= 0) {
        const double* d = sDp + 6 * slot;
        for (int c = 0; c < 3; ++c) {
          double v = 0.0;
          for (int r = 0; r < 6; ++r) v += (double)A.W[3 * r + c] * d[r];
          wtd[c] = (Real)v;
        }
      }
      for (int k = 0; k < 6; ++k) sPV[12 * q + k] = A.V[k];
      for (int k = 0; k < 3; ++k) sPV[12 * q + 6 + k] = A.gl[k];
      for (int k = 0; k < 3; ++k) sPV[12 * q + 9 + k] = wtd[k];
    }
    __syncthreads();

    // ---- phase 2: per landmark: dl = V*^-1 (c_l - sum W^T dp)
    if (tid < nL) {
      const int lmt = l0 + tid;
      const int q0 = lb0 - p0, q1 = lb1 - p0;
      Real V[6] = {0, 0, 0, 0, 0, 0}, g[3] = {0, 0, 0}, s3[3] = {0, 0, 0};
#pragma unroll 4
      for (int qq = q0; qq < q1; ++qq) {
        for (int k = 0; k < 6; ++k) V[k] += sPV[12 * qq + k];
        for (int k = 0; k < 3; ++k) g[k] += sPV[12 * qq + 6 + k];
        for (int k = 0; k < 3; ++k) s3[k] += sPV[12 * qq + 9 + k];
      }
      Real c[3];
      if (!ADJ) {
        damp3(V, lam);
        for (int k = 0; k < 3; ++k) c[k] = -g[k] - s3[k];
      } else {
        for (int k = 0; k < 3; ++k)
          c[k] = (U.grad_points ? (Real)U.grad_points[3 * lmt + k] : (Real)0) - s3[k];
      }
      LDL3<Real> F;
      ldl3(V, !ADJ, F);
      Real x[3];
      ldl3_solve(F, c, x);
      const double pt[3] = {lx, ly, lz};
      if (!ADJ) {
        double* cp = cpoints + 3 * (lmt - W.point_off);
        for (int k = 0; k < 3; ++k) {
          const double v = pt[k] + (double)x[k];
          sLP[3 * tid + k] = v;
          cp[k] = v;
          smax = fmax(smax, fabs((double)x[k]));
        }
      } else {
        for (int k = 0; k < 3; ++k) sLP[3 * tid + k] = (double)x[k];
      }
    }
    // next tile's pair records (its tile record has arrived by now)
    int4 nrec = make_int4(0, 0, 0, -1);
    if (t + 1 < t1 && tid < nta.y) nrec = prec[nta.x + tid];
    __syncthreads();
    // the next tile's pairs: points and first observations, behind phase 3
    double npx = 0, npy = 0, npz = 0;
    Real ndu = 0, ndv = 0, nwo = 1;
    int ncam = 0;
    if (t + 1 < t1 && tid < nta.y) fetch_pair(nrec, npx, npy, npz, ndu, ndv, nwo, ncam);

    // ---- phase 3: per pair: candidate cost (LM) / per-observation gradients (ADJ)
    if (tid < nP) {
      if (!ADJ) {
        const double* Rt = sPoseC + 12 * pose;
        const double* pt = sLP + 3 * j;
        double xb[3];
        for (int a = 0; a < 3; ++a)
          xb[a] = Rt[4 * a] * pt[0] + Rt[4 * a + 1] * pt[1] + Rt[4 * a + 2] * pt[2] + Rt[4 * a + 3];
        for (int o = o0; o < o0 + nobs; ++o) {
          const bool first = o == o0;   // the first observation is in registers
          const double* C = sCam + 16 * (first ? cam0 : P.obs_cam[o]);
          const double X = C[4] * xb[0] + C[5] * xb[1] + C[6] * xb[2] + C[13];
          const double Y = C[7] * xb[0] + C[8] * xb[1] + C[9] * xb[2] + C[14];
          const double Z = C[10] * xb[0] + C[11] * xb[1] + C[12] * xb[2] + C[15];
          if (!(Z > S.min_depth)) sFlag[0] = 1;
          const double iz = recip_nr(Z);
          const double r0 = C[0] * X * iz - (double)(first ? du0 : K.du[o]);
          const double r1 = C[1] * Y * iz - (double)(first ? dv0 : K.dv[o]);
          double rho, d1, d2;
          huber(r0 * r0 + r1 * r1, S.huber_delta, rho, d1, d2);
          cost += (first ? (double)wo0 : (K.w ? (double)K.w[o] : 1.0)) * rho;
        }
      } else {
        const double* Rt = sPose + 12 * pose;
        double xb[3];
        for (int a = 0; a < 3; ++a) xb[a] = Rt[4 * a] * px + Rt[4 * a + 1] * py + Rt[4 * a + 2] * pz + Rt[4 * a + 3];
        const double* al = sLP + 3 * j;
        const double zero6[6] = {0, 0, 0, 0, 0, 0};
        const double* ap = slot >= 0 ? sDp + 6 * slot : zero6;
        // R_i^T applied on the landmark part: J_l a_l = a . (R_i a_l)
        double Ral[3];
        for (int a = 0; a < 3; ++a)
          Ral[a] = Rt[4 * a] * al[0] + Rt[4 * a + 1] * al[1] + Rt[4 * a + 2] * al[2];
        // pose part: J_p a_p = a . rho + (x_b x a) . phi = a . (rho + phi x x_b)
        double pc[3];
        pc[0] = ap[4] * xb[2] - ap[5] * xb[1];
        pc[1] = ap[5] * xb[0] - ap[3] * xb[2];
        pc[2] = ap[3] * xb[1] - ap[4] * xb[0];
        double v3[3];
        for (int a = 0; a < 3; ++a) v3[a] = ap[a] + pc[a] + Ral[a];
        for (int o = o0; o < o0 + nobs; ++o) {
          const double* C = sCam + 16 * P.obs_cam[o];
          const double wo = K.w ? (double)K.w[o] : 1.0;
          const Lin<Real> L = linearise<Real>(xb, C, (double)K.du[o], (double)K.dv[o], wo,
                                              S.huber_delta);
          const double ja0 = (double)L.a0[0] * v3[0] + (double)L.a0[1] * v3[1] + (double)L.a0[2] * v3[2];
          const double ja1 = (double)L.a1[0] * v3[0] + (double)L.a1[1] * v3[1] + (double)L.a1[2] * v3[2];
          const double r0 = (double)L.r[0], r1 = (double)L.r[1];
          const double rja = r0 * ja0 + r1 * ja1;
          const int u = W.obs_off + P.obs_perm[o];
          U.grad_uv[2 * u] = wo * (L.d1 * ja0 + 2.0 * L.d2 * r0 * rja);
          U.grad_uv[2 * u + 1] = wo * (L.d1 * ja1 + 2.0 * L.d2 * r1 * rja);
          if (U.grad_w) U.grad_w[u] = -L.d1 * rja;
        }
      }
    }
    __syncthreads();
    ta = nta;
    rec = nrec;
    px = npx;
    py = npy;
    pz = npz;
    du0 = ndu;
    dv0 = ndv;
    wo0 = nwo;
    cam0 = ncam;
    lb0 = nlb0;
    lb1 = nlb1;
    lx = nlx;
    ly = nly;
    lz = nlz;
  }
  if (!ADJ) {
    const double tot = block_sum<TP>(cost, sRed);
    if (tid == 0) {
      K.part_cost_b[chunk] = tot;
      K.part_flag_b[chunk] = sFlag[0];
    }
    if (S.step_tol > 0) {
      const double sm = block_max<TP>(smax, sRed);
      if (tid == 0) K.part_smax[chunk] = sm;
    }
  }
}

// ---------------------------------------------------------------------------
// accept / finalize
// ---------------------------------------------------------------------------

template <typename Real>
__global__ void k_accept(DevPlan P, DevTiles T, DevWork<Real> K, DevUser U, DevSettings S, int it, int wbase,
                         int nwin) {
  // one wave per window
  const int i = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (i >= nwin) return;
  const WinDev W = T.win_rec[wbase + i];
  put_decision(P, K, U, S, it + 1, W.self, W.n_free, W.chunk_begin, W.chunk_end, threadIdx.x & 63);
}

// Copy the final state into the user's arrays where it sits in the workspace
// buffer, and write the report.  One workgroup per window.
template <typename Real>
__global__ void k_finalize(DevPlan P, DevWork<Real> K, DevUser U, DevSettings S, int fused) {
  const int wi = blockIdx.x;
  const WinDev W = P.win[wi];
  const int need_cost = S.max_iters == 0;
  WinState st;
  if (fused && !need_cost) {   // the last attempt's decision, by every wave
    ba_iter_trace tr;
    st = decide(state_at(P, K, S.max_iters - 1, wi), K, S, wi, W.n_free, W.chunk_begin, W.chunk_end,
                threadIdx.x & 63, tr);
    if (threadIdx.x == 0 && U.traces) U.traces[(size_t)wi * S.max_iters + S.max_iters - 1] = tr;
  } else {
    st = state_at(P, K, S.max_iters, wi);
  }
  if (st.cur == 1) {
    for (int k = threadIdx.x; k < 12 * W.n_poses; k += blockDim.x)
      U.poses[12 * W.pose_off + k] = K.poses_b[12 * W.pose_off + k];
    if (K.vi_states)
      for (int k = threadIdx.x; k < 9 * W.n_poses; k += blockDim.x)
        K.vi_states[9 * W.pose_off + k] = K.vi_states_b[9 * W.pose_off + k];
    for (int k = threadIdx.x; k < 3 * W.n_points; k += blockDim.x)
      U.points[3 * W.point_off + k] = K.points_b[3 * W.point_off + k];
  }
  // no attempt ran: the cost comes from the pass-A partials, summed as the
  // first attempt's reduce sums them
  int fdummy = 0;
  double F = 0.0;
  if (need_cost && threadIdx.x < 64)
    wave_chunk_sums(K.part_flag_a, K.part_cost_a, W.chunk_begin, W.chunk_end, true, threadIdx.x, fdummy, F);
  if (threadIdx.x == 0) {
    ba_report r;
    double c0 = st.init_cost, cf = st.cost;
    if (need_cost) c0 = cf = 0.5 * F;
    r.initial_cost = c0;
    r.final_cost = cf;
    r.final_lambda = st.lambda;
    r.iters = st.iters;
    r.accepted = st.accepted;
    r.chol_failures = st.chol_failures;
    r.depth_rejects = st.depth_rejects;
    r.status = (need_cost && !isfinite(c0)) ? 1 : st.status;
    r.reserved = 0;
    U.reports[wi] = r;
  }
}

// ---------------------------------------------------------------------------
// host-side launch helpers (instantiated here, called by the ABI layer)
// ---------------------------------------------------------------------------

template <typename Real, int TP>
size_t pass_a_lds(int np, int nc, int nf, int list_bytes, bool adj) {
  return PassALds<Real, TP>::bytes(np, nc, nf, list_bytes, adj);
}

template <typename Real, int TP>
size_t pass_b_lds() {
  return (2 * ChunkLds::kPose + ChunkLds::kCam + kDpStride + 3 * TP + 16) * sizeof(double) +
         4 * sizeof(int) + (size_t)TP * 12 * sizeof(Real);
}

// The reduce kernel's LDS: the reduced system of the largest window.
size_t reduce_lds(int max_nf) {
  const int nblk = max_nf * (max_nf + 1) / 2;
  return (size_t)(nblk * kRS + 12 * max_nf + 11) * sizeof(double);
}

constexpr int kReduceThreads = 512;

template <typename Real, int TP, bool ADJ>
hipError_t set_attrs() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pass_a<Real, TP, ADJ>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pass_b<Real, TP, ADJ>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_reduce<Real, kReduceThreads, ADJ>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

// One pass-A launch of size class c on stream st, with the LDS its largest window
// needs.
template <typename Real, bool ADJ>
void launch_pass_a_class(const LaunchArgs& A, const DevWork<Real>& K, int it, int c, hipStream_t st) {
  const int n = A.cls_begin[c + 1] - A.cls_begin[c];
  if (n <= 0) return;
  auto go = [&](auto tp) {
    constexpr int TP = decltype(tp)::value;
    const size_t lds = pass_a_lds<Real, TP>(A.dims.np, A.dims.nc, A.cls_nf[c], A.cls_list_bytes[c], ADJ);
    hipLaunchKernelGGL((k_pass_a<Real, TP, ADJ>), dim3(n), dim3(kPassAThreads), lds, st, A.plan, A.tiles, K, A.user,
                       A.settings, it, A.cls_begin[c], A.dims, A.fused);
  };
  if (A.cls_tp[c] == kTileLarge) go(std::integral_constant<int, kTileLarge>());
  else go(std::integral_constant<int, kTileSmall>());
}

// Pass A over the size classes.  With side streams, the largest class and the next
// one each run on a side stream, concurrently with the rest on the launch stream: the
// classes share the CUs, so one class's long workgroups fill the others' launch
// tails, and workgroups of a small class fit beside one of the largest class in the
// LDS of a CU (measured on the 256-window batch: +21 % LM attempts per second
// over the four launches in sequence; merging classes of equal occupancy into
// one launch gained 6 %).
template <typename Real, bool ADJ>
hipError_t launch_pass_a(const LaunchArgs& A, const DevWork<Real>& K, int it) {
  static_assert(kSideStreams >= 2, "pass A uses two side streams");
  const hipStream_t main = (hipStream_t)A.stream;
  const hipStream_t* side = (const hipStream_t*)A.side_stream;
  const hipEvent_t* join = (const hipEvent_t*)A.ev_join;
  int cls[kClasses], ng = 0;
  for (int c = 0; c < kClasses; ++c)
    if (A.cls_begin[c + 1] > A.cls_begin[c]) cls[ng++] = c;
  const int nside = A.side_stream && ng >= 2 ? (ng >= 3 ? 2 : 1) : 0;   // the largest nside classes
  hipError_t e = hipSuccess;
  if (nside && (e = hipEventRecord((hipEvent_t)A.ev_fork, main)) != hipSuccess) return e;
  for (int s = 0; s < nside; ++s) {   // side launches first
    if ((e = hipStreamWaitEvent(side[s], (hipEvent_t)A.ev_fork, 0)) != hipSuccess) return e;
    launch_pass_a_class<Real, ADJ>(A, K, it, cls[ng - 1 - s], side[s]);
  }
  for (int k = 0; k < ng - nside; ++k) launch_pass_a_class<Real, ADJ>(A, K, it, cls[k], main);
  for (int s = 0; s < nside; ++s) {
    if ((e = hipEventRecord(join[s], side[s])) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(main, join[s], 0)) != hipSuccess) return e;
  }
  return hipGetLastError();
}

// Pass B over the chunks of the size classes [ca, cb): neighbouring classes of one
// tile size share a launch.
template <typename Real, bool ADJ>
void launch_pass_b(const LaunchArgs& A, const DevWork<Real>& K, int it, int ca, int cb, hipStream_t st) {
  for (int c = ca; c < cb;) {
    int d = c + 1;
    while (d < cb && A.cls_tp[d] == A.cls_tp[c]) ++d;
    const int n = A.cls_begin[d] - A.cls_begin[c];
    auto go = [&](auto tp) {
      constexpr int TP = decltype(tp)::value;
      const size_t lds = pass_b_lds<Real, TP>();
      hipLaunchKernelGGL((k_pass_b<Real, TP, ADJ>), dim3(n), dim3(TP), lds, st, A.plan, A.tiles, K, A.user, A.settings,
                         it, A.cls_begin[c]);
    };
    if (n > 0) {
      if (A.cls_tp[c] == kTileLarge) go(std::integral_constant<int, kTileLarge>());
      else go(std::integral_constant<int, kTileSmall>());
    }
    c = d;
  }
}

// The stages after pass A of one LM attempt for the windows of the size classes
// [ca, cb) (at most nf free poses each) on stream st.
template <typename Real, bool ADJ>
void launch_stages(const LaunchArgs& A, const DevWork<Real>& K, int it, int ca, int cb, int nf, int slices,
                   hipStream_t st) {
  const int wb = A.cls_win_begin[ca], nwin = A.cls_win_begin[cb] - wb;
  if (nwin <= 0) return;
  const size_t lr = reduce_lds(nf);
  hipLaunchKernelGGL(k_sum<Real>, dim3(nwin, slices), dim3(256), 0, st, A.plan, A.tiles, K, A.user, A.settings, it, wb,
                     A.fused);
  ViArgs V;
  if (!ADJ && A.vi) {
    V = *static_cast<const ViArgs*>(A.vi);
    V.state += (it & 1) * A.plan.n_windows;
    launch_vi_lin(V, wb, nwin, st);
  }
  hipLaunchKernelGGL((k_reduce<Real, kReduceThreads, ADJ>), dim3(nwin), dim3(kReduceThreads), lr, st, A.plan, A.tiles,
                     K, A.user, A.settings, it, wb);
  if (!ADJ && A.vi) launch_vi_cand(V, wb, nwin, st);
  launch_pass_b<Real, ADJ>(A, K, it, ca, cb, st);
  if (!ADJ && !A.fused)
    hipLaunchKernelGGL(k_accept<Real>, dim3((nwin + 3) / 4), dim3(256), 0, st, A.plan, A.tiles, K, A.user,
                       A.settings, it, wb, nwin);
}

// The windows of one size class never meet those of another, so with side
// streams every class runs its whole LM loop (pass A, sum, reduce, pass B,
// acceptance per attempt) as a chain of its own, forked once after the set-up
// and joined once before the final copy: the largest class on side stream 1,
// the next on side stream 2, the smaller ones one after the other on the
// launch stream (as pass A's split in launch_pass_a).  The small grids of the
// reduce and pass B then overlap with other classes' pass A instead of every
// class waiting for the slowest one in each attempt (256-window batch: 271 k
// -> 285 k LM attempts/s; four chains on four streams: 279 k; the smallest
// class on a side stream with a larger one: 242-273 k).
struct ClassChains {
  int n = 0, nside = 0;
  int cls[kClasses];            // the classes that hold windows, ascending
  hipStream_t st[kClasses];     // the stream of each
};

// The chains of a launch, or n = 0 when everything runs on the launch stream
// (no side streams, or fewer than two classes).
inline ClassChains class_chains(const LaunchArgs& A) {
  ClassChains C;
  int ncls = 0;
  for (int c = 0; c < kClasses; ++c)
    if (A.cls_win_begin[c + 1] > A.cls_win_begin[c]) C.cls[ncls++] = c;
  if (!A.side_stream || ncls < 2) return C;
  const hipStream_t* side = (const hipStream_t*)A.side_stream;
  C.n = ncls;
  C.nside = ncls >= 3 ? 2 : 1;   // classes on side streams: the largest nside
  for (int k = 0; k < ncls; ++k) {
    const int r = ncls - 1 - k;  // rank from the largest class
    C.st[k] = r < C.nside ? side[r] : (hipStream_t)A.stream;
  }
  return C;
}

inline hipError_t fork_chains(const LaunchArgs& A, const ClassChains& C) {
  const hipStream_t* side = (const hipStream_t*)A.side_stream;
  hipError_t e = hipEventRecord((hipEvent_t)A.ev_fork, (hipStream_t)A.stream);
  for (int r = 0; r < C.nside && e == hipSuccess; ++r) e = hipStreamWaitEvent(side[r], (hipEvent_t)A.ev_fork, 0);
  return e;
}

inline hipError_t join_chains(const LaunchArgs& A, const ClassChains& C) {
  const hipStream_t* side = (const hipStream_t*)A.side_stream;
  const hipEvent_t* join = (const hipEvent_t*)A.ev_join;
  hipError_t e = hipSuccess;
  for (int r = 0; r < C.nside && e == hipSuccess; ++r) {
    e = hipEventRecord(join[r], side[r]);
    if (e == hipSuccess) e = hipStreamWaitEvent((hipStream_t)A.stream, join[r], 0);
  }
  return e;
}

// One attempt of class C.cls[k] on its chain's stream.
template <typename Real, bool ADJ>
void launch_class_attempt(const LaunchArgs& A, const DevWork<Real>& K, int it, const ClassChains& C, int k) {
  const int c = C.cls[k];
  launch_pass_a_class<Real, ADJ>(A, K, it, c, C.st[k]);
  launch_stages<Real, ADJ>(A, K, it, c, c + 1, A.cls_win_nf[c], A.cls_sum_slices[c], C.st[k]);
}

template <typename Real>
hipError_t run_solve(const LaunchArgs& A, const DevWork<Real>& K) {
  const int nw = A.plan.n_windows, nc = A.tiles.n_chunks;
  const hipStream_t main = (hipStream_t)A.stream;
  hipLaunchKernelGGL(k_init<Real>, dim3((nw + 63) / 64), dim3(64), 0, main, A.plan, K, A.settings);
  hipLaunchKernelGGL(k_pack<Real>, dim3(nc), dim3(256), 0, main, A.plan, A.tiles, K, A.user);
  const int iters = A.settings.max_iters;
  const ClassChains C = class_chains(A);
  hipError_t e = hipSuccess;
  if (C.n > 0 && iters > 0) {
    if ((e = fork_chains(A, C)) != hipSuccess) return e;
    for (int it = 0; it < iters; ++it)
      for (int k = C.n - 1; k >= 0; --k) launch_class_attempt<Real, false>(A, K, it, C, k);
    if ((e = join_chains(A, C)) != hipSuccess) return e;
  } else {
    for (int it = 0; it < iters; ++it) {
      if ((e = launch_pass_a<Real, false>(A, K, it)) != hipSuccess) return e;
      launch_stages<Real, false>(A, K, it, 0, kClasses, A.max_nf, A.sum_slices, main);
    }
  }
  if (iters == 0 && (e = launch_pass_a<Real, false>(A, K, 0)) != hipSuccess)   // the report still needs the input cost
    return e;
  hipLaunchKernelGGL(k_finalize<Real>, dim3(nw), dim3(256), 0, main, A.plan, K, A.user, A.settings, A.fused);
  return hipGetLastError();
}

// The adjoint's single pass, in the same class chains as a solve.
template <typename Real>
hipError_t run_adjoint(const LaunchArgs& A, const DevWork<Real>& K) {
  const int nw = A.plan.n_windows, nc = A.tiles.n_chunks;
  const hipStream_t main = (hipStream_t)A.stream;
  hipLaunchKernelGGL(k_init<Real>, dim3((nw + 63) / 64), dim3(64), 0, main, A.plan, K, A.settings);
  hipLaunchKernelGGL(k_pack<Real>, dim3(nc), dim3(256), 0, main, A.plan, A.tiles, K, A.user);
  const ClassChains C = class_chains(A);
  hipError_t e = hipSuccess;
  if (C.n > 0) {
    if ((e = fork_chains(A, C)) != hipSuccess) return e;
    for (int k = C.n - 1; k >= 0; --k) launch_class_attempt<Real, true>(A, K, 0, C, k);
    if ((e = join_chains(A, C)) != hipSuccess) return e;
  } else {
    if ((e = launch_pass_a<Real, true>(A, K, 0)) != hipSuccess) return e;
    launch_stages<Real, true>(A, K, 0, 0, kClasses, A.max_nf, A.sum_slices, main);
  }
  return hipGetLastError();
}

// The attempt-by-attempt sequence (pass A's classes forked and joined within
// each attempt, the other stages over all windows on the launch stream) with
// HIP events between the stages: the summed device time of each stage
// (pass_a, reduce, pass_b, accept) in ms, for the roofline figures of the
// benchmark.  Synchronises on the stream.
template <typename Real>
hipError_t run_solve_timed(const LaunchArgs& A, const DevWork<Real>& K, double* stage_ms) {
  const int nw = A.plan.n_windows, nc = A.tiles.n_chunks;
  const hipStream_t main = (hipStream_t)A.stream;
  const size_t lr = reduce_lds(A.max_nf);
  const int iters = A.settings.max_iters;
  const int nev = 4 * iters + 1;
  hipEvent_t* ev = new hipEvent_t[nev];
  for (int k = 0; k < nev; ++k) (void)hipEventCreate(&ev[k]);
  hipLaunchKernelGGL(k_init<Real>, dim3((nw + 63) / 64), dim3(64), 0, main, A.plan, K, A.settings);
  hipLaunchKernelGGL(k_pack<Real>, dim3(nc), dim3(256), 0, main, A.plan, A.tiles, K, A.user);
  (void)hipEventRecord(ev[0], main);
  hipError_t e = hipSuccess;
  for (int it = 0; it < iters && e == hipSuccess; ++it) {
    e = launch_pass_a<Real, false>(A, K, it);
    (void)hipEventRecord(ev[4 * it + 1], main);
    hipLaunchKernelGGL(k_sum<Real>, dim3(nw, A.sum_slices), dim3(256), 0, main, A.plan, A.tiles, K, A.user,
                       A.settings, it, 0, 0);
    hipLaunchKernelGGL((k_reduce<Real, kReduceThreads, false>), dim3(nw), dim3(kReduceThreads), lr, main, A.plan,
                       A.tiles, K, A.user, A.settings, it, 0);
    (void)hipEventRecord(ev[4 * it + 2], main);
    launch_pass_b<Real, false>(A, K, it, 0, kClasses, main);
    (void)hipEventRecord(ev[4 * it + 3], main);
    hipLaunchKernelGGL(k_accept<Real>, dim3((nw + 3) / 4), dim3(256), 0, main, A.plan, A.tiles, K, A.user,
                       A.settings, it, 0, nw);
    (void)hipEventRecord(ev[4 * it + 4], main);
  }
  hipLaunchKernelGGL(k_finalize<Real>, dim3(nw), dim3(256), 0, main, A.plan, K, A.user, A.settings, 0);
  if (e == hipSuccess) e = hipGetLastError();
  if (e == hipSuccess) e = hipEventSynchronize(ev[nev - 1]);
  for (int k = 0; k < 4; ++k) stage_ms[k] = 0.0;
  for (int it = 0; it < iters && e == hipSuccess; ++it)
    for (int k = 0; k < 4; ++k) {
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, ev[4 * it + k], ev[4 * it + k + 1]);
      stage_ms[k] += ms;
    }
  for (int k = 0; k < nev; ++k) (void)hipEventDestroy(ev[k]);
  delete[] ev;
  return e;
}

// explicit instantiations used by the ABI layer
template size_t pass_a_lds<double, 64>(int, int, int, int, bool);
template size_t pass_a_lds<double, 256>(int, int, int, int, bool);
template size_t pass_a_lds<float, 64>(int, int, int, int, bool);
template size_t pass_a_lds<float, 256>(int, int, int, int, bool);
template size_t pass_b_lds<double, 64>();
template size_t pass_b_lds<double, 256>();
template size_t pass_b_lds<float, 64>();
template size_t pass_b_lds<float, 256>();
template hipError_t set_attrs<double, 64, false>();
template hipError_t set_attrs<double, 256, false>();
template hipError_t set_attrs<float, 64, false>();
template hipError_t set_attrs<float, 256, false>();
template hipError_t set_attrs<double, 64, true>();
template hipError_t set_attrs<double, 256, true>();
template hipError_t set_attrs<float, 64, true>();
template hipError_t set_attrs<float, 256, true>();
template hipError_t run_solve<double>(const LaunchArgs&, const DevWork<double>&);
template hipError_t run_solve<float>(const LaunchArgs&, const DevWork<float>&);
template hipError_t run_solve_timed<double>(const LaunchArgs&, const DevWork<double>&, double*);
template hipError_t run_solve_timed<float>(const LaunchArgs&, const DevWork<float>&, double*);
template hipError_t run_adjoint<double>(const LaunchArgs&, const DevWork<double>&);
template hipError_t run_adjoint<float>(const LaunchArgs&, const DevWork<float>&);

}  // namespace ba
