// gfx950 pose-graph optimisation (paper Sec. 2.3, Eq. 15): LM over the
// world-from-base poses T_i minimising 1/2 sum_e w_e |Log(D_ij^-1 T_i^-1 T_j)|^2.
//
// Per LM attempt:
//   k_pgo_edges  one thread per edge at the candidate poses: r = Log(E),
//                E = D^-1 T_i^-1 T_j, B = J_l(r)^-1 Ad(D^-1 T_i^-1) (so dr/dxi_j
//                = B, dr/dxi_i = -B for the left perturbation), and w B^T B,
//                w B^T r, w |r|^2 into an edge buffer (two buffers: the current
//                linearisation and the candidate's)
//   k_pgo_decide     one workgroup: the candidate's cost (fixed-order sum),
//                    accept iff it strictly drops, lambda, trace
//   k_pgo_assemble   the damped normal equations gathered from the current
//                    edge buffer into the factor's blocks, -g into y
//   k_pgo_tree       the sparse block Cholesky, one launch per tier of the
//                    elimination tree (left-looking: each column gathers its
//                    updates, factors its diagonal block in registers, solves its
//                    panel; the forward substitution rides along); the last tier's
//                    one workgroup starts the back substitution
//   k_pgo_back       the back substitution of the earlier tiers
//   k_pgo_candidate  the next candidate Exp(d_i) T_i
// Every sum has a fixed order and nothing uses atomics.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "device.hpp"
#include "geometry.hpp"
#include "pgo.hpp"

namespace ba {

constexpr int kPgoEdgeThreads = 256;
constexpr int kPgoStepThreads = 1024;

// 3x3 helpers (row-major)
__device__ __forceinline__ void mm3(const double* A, const double* B, double* C) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) C[3 * a + b] = A[3 * a] * B[b] + A[3 * a + 1] * B[3 + b] + A[3 * a + 2] * B[6 + b];
}
__device__ __forceinline__ void skew3(const double* v, double* K) {
  K[0] = 0.0; K[1] = -v[2]; K[2] = v[1];
  K[3] = v[2]; K[4] = 0.0; K[5] = -v[0];
  K[6] = -v[1]; K[7] = v[0]; K[8] = 0.0;
}
// C = A B for 3x4 transforms; inverse of a 3x4 transform
__device__ __forceinline__ void tcompose(const double* A, const double* B, double* C) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int b = 0; b < 3; ++b) C[4 * a + b] = A[4 * a] * B[b] + A[4 * a + 1] * B[4 + b] + A[4 * a + 2] * B[8 + b];
    C[4 * a + 3] = A[4 * a] * B[3] + A[4 * a + 1] * B[7] + A[4 * a + 2] * B[11] + A[4 * a + 3];
  }
}
__device__ __forceinline__ void tinverse(const double* T, double* I) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int b = 0; b < 3; ++b) I[4 * a + b] = T[4 * b + a];
    I[4 * a + 3] = -(T[a] * T[3] + T[4 + a] * T[7] + T[8 + a] * T[11]);
  }
}

// Log of a rotation: phi with Exp(phi) = R.  theta = atan2(|v|, (tr R - 1) / 2)
// with v the vee of the antisymmetric part (sin(theta) times the axis); the
// axis from the symmetric part near theta = pi.
__device__ __forceinline__ void log_so3(const double* T /*3x4*/, double* phi) {
  const double v[3] = {0.5 * (T[9] - T[6]), 0.5 * (T[2] - T[8]), 0.5 * (T[4] - T[1])};
  double c = 0.5 * (T[0] + T[5] + T[10] - 1.0);
  c = fmin(1.0, fmax(-1.0, c));
  const double s = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  const double th = atan2(s, c);
  if (c > -0.999) {
    // theta / sin(theta); series below theta = 1e-3
    const double t2 = th * th;
    const double f = th < 1e-3 ? 1.0 + t2 * (1.0 / 6.0 + t2 * (7.0 / 360.0)) : th / s;
    phi[0] = f * v[0];
    phi[1] = f * v[1];
    phi[2] = f * v[2];
    return;
  }
  // (R + R^T) / 2 = c I + (1 - c) a a^T
  const double Md[3] = {T[0] - c, T[5] - c, T[10] - c};
  int k = 0;
  if (Md[1] > Md[k]) k = 1;
  if (Md[2] > Md[k]) k = 2;
  const double ic = 1.0 / (1.0 - c);
  double a[3];
  a[k] = sqrt(fmax(Md[k] * ic, 0.0));
  const double ia = 1.0 / a[k];
#pragma unroll
  for (int m = 0; m < 3; ++m)
    if (m != k) a[m] = 0.5 * (T[4 * m + k] + T[4 * k + m]) * ic * ia;
  const double sg = (a[0] * v[0] + a[1] * v[1] + a[2] * v[2]) < 0.0 ? -1.0 : 1.0;
  phi[0] = sg * th * a[0];
  phi[1] = sg * th * a[1];
  phi[2] = sg * th * a[2];
}

// Inverse of the SO(3) left Jacobian: I - K/2 + d K^2, d = 1/th^2 -
// cot(th/2) / (2 th) (series below th = 0.1).
__device__ __forceinline__ void jl_inv_so3(const double* phi, double* Ji) {
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
  mm3(K, K, K2);
#pragma unroll
  for (int k = 0; k < 9; ++k) Ji[k] = ((k % 4 == 0) ? 1.0 : 0.0) - 0.5 * K[k] + d * K2[k];
}

// Top-right block Q of the SE(3) left Jacobian J_l(rho, phi) =
// sum_n ad^n / (n+1)!: with ad^n = [[K^n, X_n], [0, K^n]], X_{n+1} = K X_n +
// P K^n (P = rho^), Q = sum_{n >= 1} X_n / (n+1)!; summed until the bound
// th^n n |rho| / (n+1)! is below 1e-18 (at most 40 terms).
__device__ __forceinline__ void jl_q_se3(const double* rho, const double* phi, double* Q) {
  double K[9], P[9], Kn[9], X[9], t1[9], t2[9];
  skew3(phi, K);
  skew3(rho, P);
  const double th = sqrt(phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2]);
  const double nr = sqrt(rho[0] * rho[0] + rho[1] * rho[1] + rho[2] * rho[2]);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    Kn[k] = (k % 4 == 0) ? 1.0 : 0.0;   // K^0
    X[k] = 0.0;                          // X_0
    Q[k] = 0.0;
  }
  double fact = 1.0;    // (n+1)!
  double thn = 1.0;     // th^n
  for (int n = 0; n < 40; ++n) {
    // X_{n+1} = K X_n + P K^n, K^{n+1} = K K^n
    mm3(K, X, t1);
    mm3(P, Kn, t2);
#pragma unroll
    for (int k = 0; k < 9; ++k) X[k] = t1[k] + t2[k];
    mm3(K, Kn, t1);
#pragma unroll
    for (int k = 0; k < 9; ++k) Kn[k] = t1[k];
    fact *= (double)(n + 2);   // (n+2)!
#pragma unroll
    for (int k = 0; k < 9; ++k) Q[k] += X[k] / fact;
    thn *= th;
    if (thn * (n + 1) * nr / fact < 1e-18 && n >= 1) break;
  }
}

__global__ __launch_bounds__(kPgoEdgeThreads) void k_pgo_edges(PgoArgs A, int init) {
  const int e = blockIdx.x * kPgoEdgeThreads + threadIdx.x;
  if (e >= A.G.n_edges) return;
  const int cur = A.W.istate[0];
  double* out = A.W.edge[init ? 0 : 1 - cur] + 28 * (long long)e;
  const double* P = init ? A.poses : A.W.cand;
  const double* Ti = P + 12 * (long long)A.G.edge_i[e];
  const double* Tj = P + 12 * (long long)A.G.edge_j[e];
  const double* D = A.deltas + 12 * (long long)e;
  const double w = A.edge_w ? A.edge_w[e] : 1.0;
  double Di[12], Tii[12], X[12], E[12];
  tinverse(D, Di);
  tinverse(Ti, Tii);
  tcompose(Di, Tii, X);   // D^-1 T_i^-1
  tcompose(X, Tj, E);     // D^-1 T_i^-1 T_j
  // r = Log(E) = (J^-1 t, phi)
  double phi[3], Ji[9], r[6];
  log_so3(E, phi);
  jl_inv_so3(phi, Ji);
#pragma unroll
  for (int a = 0; a < 3; ++a) r[a] = Ji[3 * a] * E[3] + Ji[3 * a + 1] * E[7] + Ji[3 * a + 2] * E[11];
  r[3] = phi[0];
  r[4] = phi[1];
  r[5] = phi[2];
  // B = J_l(r)^-1 Ad(X) = [[M, N], [0, M]]: M = J^-1 R_X, N = J^-1 (t_X^ R_X - Q M)
  double Q[9], R[9], M[9], tX[9], K1[9], QM[9], N[9], tmp[9];
  jl_q_se3(r, phi, Q);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) R[3 * a + b] = X[4 * a + b];
  mm3(Ji, R, M);
  const double tv[3] = {X[3], X[7], X[11]};
  skew3(tv, tX);
  mm3(tX, R, K1);
  mm3(Q, M, QM);
#pragma unroll
  for (int k = 0; k < 9; ++k) tmp[k] = K1[k] - QM[k];
  mm3(Ji, tmp, N);
  // B (6x6) explicitly, then w B^T B (upper), w B^T r, w |r|^2
  double B[36];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      B[6 * a + b] = M[3 * a + b];
      B[6 * a + 3 + b] = N[3 * a + b];
      B[6 * (a + 3) + b] = 0.0;
      B[6 * (a + 3) + 3 + b] = M[3 * a + b];
    }
  int k = 0;
#pragma unroll
  for (int a = 0; a < 6; ++a)
#pragma unroll
    for (int b = a; b < 6; ++b, ++k) {
      double v = 0.0;
#pragma unroll
      for (int m = 0; m < 6; ++m) v += B[6 * m + a] * B[6 * m + b];
      out[k] = w * v;
    }
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    double v = 0.0;
#pragma unroll
    for (int m = 0; m < 6; ++m) v += B[6 * m + a] * r[m];
    out[21 + a] = w * v;
  }
  double rr = 0.0;
#pragma unroll
  for (int m = 0; m < 6; ++m) rr += r[m] * r[m];
  out[27] = w * rr;
}

// upper-triangle index of (a, b) in a 6x6 symmetric block
__device__ __forceinline__ int up6(int a, int b) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  return 6 * lo - lo * (lo - 1) / 2 + hi - lo;
}

// Decision on the candidate just evaluated (mode 1), or the start (mode 0):
// the cost summed in a fixed order, accept iff it strictly drops, lambda,
// trace, the accepted poses, and the report after the last attempt.
__global__ __launch_bounds__(kPgoStepThreads) void k_pgo_decide(PgoArgs A, int mode, int it, int last) {
  __shared__ double sRed[kPgoStepThreads];
  const int tid = threadIdx.x;
  const PgoDev& G = A.G;
  const PgoWork& W = A.W;
  const DevSettings S = A.settings;
  double* st = W.state;      // 0 F, 1 lambda, 2 F0
  int32_t* ist = W.istate;   // 0 current buffer, 1 candidate valid, 2 accepted, 3 chol failures
  const int cur0 = mode == 0 ? 0 : ist[0];
  const int ev = mode == 0 ? 0 : 1 - cur0;
  double s = 0.0;
  for (int e = tid; e < G.n_edges; e += kPgoStepThreads) s += W.edge[ev][28 * (long long)e + 27];
  // halving tree over the threads, from 64 partial sums on within a wave: with a barrier
  // per halving and the poses' copy here the launch took 9.8 us at 3k edges, now 5.9
  sRed[tid] = s;
  __syncthreads();
  if (tid < 64) {
    double v[kPgoStepThreads / 64];
#pragma unroll
    for (int k = 0; k < kPgoStepThreads / 64; ++k) v[k] = sRed[tid + 64 * k];
#pragma unroll
    for (int h = kPgoStepThreads / 128; h > 0; h >>= 1)
#pragma unroll
      for (int k = 0; k < h; ++k) v[k] += v[k + h];
    const double t = wave_sum(v[0]);
    if (tid == 0) sRed[0] = t;
  }
  __syncthreads();
  const double Fe = 0.5 * sRed[0];
  double F, lam;
  if (mode == 0) {
    F = Fe;
    lam = S.lambda_init;
    if (tid == 0) {
      st[0] = F;
      st[1] = lam;
      st[2] = F;
      ist[0] = 0;
      ist[2] = 0;
      ist[3] = 0;
      ist[5] = 0;
    }
  } else {
    F = st[0];
    lam = st[1];
    const bool valid = ist[1] != 0;
    const bool accept = valid && Fe < F;
    if (tid == 0 && A.traces) {
      ba_iter_trace tr;
      tr.cost = F;
      tr.lambda = lam;
      tr.cand_cost = valid ? Fe : __builtin_nan("");
      tr.status = valid ? 0 : 1;
      tr.accepted = accept ? 1 : 0;
      A.traces[it] = tr;
    }
    if (accept) {
      // the accepted poses, here after the last attempt and otherwise by the assembly
      if (last)
        for (int k = tid; k < 12 * G.n_poses; k += kPgoStepThreads) A.poses[k] = W.cand[k];
      F = Fe;
    }
    lam = accept ? fmax(lam / S.lambda_down, S.lambda_min) : fmin(lam * S.lambda_up, S.lambda_max);
    if (tid == 0) {
      st[0] = F;
      st[1] = lam;
      ist[5] = accept ? 1 : 0;
      if (accept) {
        ist[0] = 1 - cur0;
        ist[2] += 1;
      }
    }
  }
  if (last && tid == 0 && A.report) {
    ba_report r;
    r.initial_cost = mode == 0 ? F : st[2];
    r.final_cost = F;
    r.final_lambda = lam;
    r.iters = S.max_iters;
    r.accepted = mode == 0 ? 0 : ist[2];
    r.chol_failures = mode == 0 ? 0 : ist[3];
    r.depth_rejects = 0;
    r.status = isfinite(r.initial_cost) ? 0 : 1;
    r.reserved = 0;
    *A.report = r;
  }
}

// The damped normal equations gathered from the current edge buffer into the
// factor's blocks (one thread per block row), and -g into y.
__global__ __launch_bounds__(kPgoEdgeThreads) void k_pgo_assemble(PgoArgs A) {
  const PgoDev& G = A.G;
  const PgoWork& W = A.W;
  const int t = blockIdx.x * kPgoEdgeThreads + threadIdx.x;
  const double* EB = W.edge[W.istate[0]];
  if (W.istate[5])   // the last attempt's poses were accepted
    for (int k = t; k < 12 * G.n_poses; k += gridDim.x * kPgoEdgeThreads) A.poses[k] = W.cand[k];
  if (t == 0) W.istate[4] = 0;   // pivot failure flag of the factorisation that follows
  const int nb6 = G.n_blocks * 6;
  if (t < nb6) {
    const int b = t / 6, a = t % 6;
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int q = G.asm_ptr[b]; q < G.asm_ptr[b + 1]; ++q) {
      const int ce = G.asm_edge[q];
      const double* x = EB + 28 * (long long)(ce >> 1);
      const double sg = (ce & 1) ? -1.0 : 1.0;
#pragma unroll
      for (int c = 0; c < 6; ++c) v[c] += sg * x[up6(a, c)];
    }
    if (G.blk_ptr[G.blk_row[b]] == b) {   // diagonal block: damping
      const double lam = W.state[1];
      v[a] += lam * fmax(v[a], 1e-9);
    }
    double* out = W.L + 36 * (long long)b + 6 * a;
#pragma unroll
    for (int c = 0; c < 6; ++c) out[c] = v[c];
  } else if (t < nb6 + G.n_free) {
    const int c = t - nb6;
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int q = G.rhs_ptr[c]; q < G.rhs_ptr[c + 1]; ++q) {
      const int ce = G.rhs_edge[q];
      const double* x = EB + 28 * (long long)(ce >> 1) + 21;
      const double sg = (ce & 1) ? -1.0 : 1.0;
#pragma unroll
      for (int a = 0; a < 6; ++a) v[a] += sg * x[a];
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) W.y[6 * c + a] = v[a];
  }
}

// Sparse block Cholesky by tiers of the elimination tree (see PgoPlan): a tier is one
// launch, a workgroup per group of subtrees, which it works through step by step (a
// step: columns of one level).  Per step: (1) every chunk of at most kPgoChunk
// updates L_rk L_ck^T of a block (and of forward updates L_ck y_k of a right-hand
// side) is summed by its own thread into a partial in LDS; (2) the partials are
// subtracted in chunk order, one entry per thread; (3) one wave per column factors the
// diagonal block in registers and solves the panel's rows and the right-hand side's.
// Back substitution tier by tier from the top.  A failed pivot sets istate[4].
//
// The solve is a chain of 33 levels (1500-pose helix), each a few dependent steps:
// latency bounds it.  With a launch per level for the lower 21 (10 us each: a chain of
// index reads, partials through memory) and one workgroup for the narrow levels
// above and the whole back substitution (287 us) an attempt's factorisation took 498 us;
// with the step's records read in one go, partials and blocks in LDS, four tiers and
// the back substitution in the same groups it takes 254 us.  Same sums in the same
// order.
// A column too large for a step: its partials go through memory.  Phase (1) over all its
// chunks: per update chunk four tasks, of 3 x 3 entries each, per forward chunk six.
// One entry per task reads three times as much.  With that, the rows of the panel solved
// by one wave and the column's back substitution by six lanes, an attempt took 4.55 ms on
// a complete graph of 80 poses and 59 ms on a chain of 1500 with 300 random closures;
// now 1.91 and 23.7 ms.
__device__ __forceinline__ void pgo_big_sums(const PgoDev& G, const PgoWork& W, int c, int bd, int n, int t0,
                                             int stride) {
  double* fpart = W.part + 36 * (long long)G.n_chunks;
  const int q0 = G.chunk_ptr[bd], nq = (G.chunk_ptr[bd + n] - q0) * 4;
  const int f0 = G.fchunk_ptr[c], nf = (G.fchunk_ptr[c + 1] - f0) * 6;
  for (int t = t0; t < nq + nf; t += stride) {
    if (t < nq) {
      const long long q = q0 + t / 4;
      const int32_t* ab = G.chunk_ab + 2 * kPgoChunk * q;
      const int r0 = (t & 2) ? 3 : 0, c0 = (t & 1) ? 3 : 0;
      double acc[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) acc[e] = 0.0;
#pragma unroll 2
      for (int k = 0; k < kPgoChunk; ++k) {
        const int ia = ab[k], ib = ab[kPgoChunk + k];
        const bool on = ia >= 0;
        const double* La = W.L + 36 * (long long)max(ia, 0) + 6 * r0;
        const double* Lb = W.L + 36 * (long long)max(ib, 0) + 6 * c0;
        double la[18], lb[18];
#pragma unroll
        for (int m = 0; m < 18; ++m) {
          la[m] = La[m];
          lb[m] = Lb[m];
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) {
          double s = 0.0;
#pragma unroll
          for (int m = 0; m < 6; ++m) s += la[6 * (e / 3) + m] * lb[6 * (e % 3) + m];
          acc[e] += on ? s : 0.0;
        }
      }
      double* out = W.part + 36 * q + 6 * r0 + c0;
#pragma unroll
      for (int e = 0; e < 9; ++e) out[6 * (e / 3) + e % 3] = acc[e];
    } else {
      const int u = t - nq, a = u % 6;
      const long long fq = f0 + u / 6;
      const int32_t* bc = G.fchunk_bc + 2 * kPgoChunk * fq;
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < kPgoChunk; ++k) {
        const int ib = bc[k], ik = bc[kPgoChunk + k];
        const double* Lf = W.L + 36 * (long long)max(ib, 0) + 6 * a;
        const double* yk = W.y + 6 * max(ik, 0);
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < 6; ++m) s += Lf[m] * yk[m];
        acc += ib >= 0 ? s : 0.0;
      }
      fpart[6 * fq + a] = acc;
    }
  }
}

// v minus p[0], p[stride], ..., p[(n - 1) stride] in order, eight reads in flight.
__device__ __forceinline__ double minus_list(double v, const double* p, int stride, int n) {
  for (int q = 0; q < n; q += 8) {
    double x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = p[(long long)stride * min(q + j, n - 1)];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (q + j < n) v -= x[j];
  }
  return v;
}

// Phase (2) of a large column c: its partials subtracted from its blocks and right-hand
// side, one entry per thread, in chunk order.
__device__ __forceinline__ void pgo_big_subtract(const PgoDev& G, const PgoWork& W, int c, int bd, int n, int t0,
                                                 int stride) {
  const double* fpart = W.part + 36 * (long long)G.n_chunks;
  for (int t = t0; t < n * 36 + 6; t += stride) {
    if (t < n * 36) {
      const int b = bd + t / 36, e = t % 36, q0 = G.chunk_ptr[b];
      double* L = W.L + 36 * (long long)b + e;
      *L = minus_list(*L, W.part + 36 * (long long)q0 + e, 36, G.chunk_ptr[b + 1] - q0);
    } else {
      const int a = t - n * 36, f0 = G.fchunk_ptr[c];
      W.y[6 * c + a] = minus_list(W.y[6 * c + a], fpart + 6 * (long long)f0 + a, 6, G.fchunk_ptr[c + 1] - f0);
    }
  }
}

// Cholesky of a 6x6 block in registers (lower part), the same in every lane.
__device__ __forceinline__ bool pgo_chol6(double (&m)[36]) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double d = m[7 * k];
#pragma unroll
    for (int q = 0; q < k; ++q) d -= m[6 * k + q] * m[6 * k + q];
    ok = ok && d > 0.0 && isfinite(d);
    const double lk = sqrt(fmax(d, 1e-300)), il = 1.0 / lk;
    m[7 * k] = lk;
#pragma unroll
    for (int i = k + 1; i < 6; ++i) {
      double v = m[6 * i + k];
#pragma unroll
      for (int q = 0; q < k; ++q) v -= m[6 * i + q] * m[6 * k + q];
      m[6 * i + k] = v * il;
    }
  }
  return ok;
}

// Factors the diagonal block at blk (its updates subtracted) in registers, the same in
// every lane, and solves rows t0, t0 + stride, ... of the column's blocks behind it (36
// per block) and of rhs, which is one more row, into the factor and y.  A pivot failure
// is raised instead.
__device__ __forceinline__ bool pgo_rows(const PgoWork& W, int c, int bd, int nblk, const double* blk,
                                         const double* rhs, int t0, int stride, int* sfail, double (&m)[36]) {
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int k = 0; k <= i; ++k) m[6 * i + k] = blk[6 * i + k];
  if (!pgo_chol6(m)) {
    if (t0 == 0) {
      W.istate[4] = 1;
      *sfail = 1;
    }
    return false;
  }
  const int nrow = (nblk - 1) * 6;
  for (int t = t0; t <= nrow; t += stride) {
    const double* row = t < nrow ? blk + 36 + 6 * t : rhs;
    double* out = t < nrow ? W.L + 36 * (long long)(bd + 1) + 6 * t : W.y + 6 * c;
    double x[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) x[k] = row[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      double v = x[k];
#pragma unroll
      for (int q = 0; q < k; ++q) v -= x[q] * m[6 * k + q];
      x[k] = v / m[7 * k];
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) out[k] = x[k];
  }
  return true;
}
__device__ __forceinline__ void pgo_store_diag(const PgoWork& W, int bd, const double (&m)[36]) {
  double* Lc = W.L + 36 * (long long)bd;
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int k = 0; k <= i; ++k) Lc[6 * i + k] = m[6 * i + k];
}

constexpr int kTreeThreads = 512;

struct TreeLds {
  double part[kStepChunks * kPgoChunk * 36];   // a chunk's products, pair by pair
  double fwd[kStepFwd * kPgoChunk * 6];
  double blk[kStepBlks * 36];   // blocks, updates subtracted; back substitution: a block's products
  double rhs[kStepCols * 6];
  double v[kTreeThreads];
  int fail;
};

// What a thread reads of a step before it can start, nothing of it written by the
// steps before, in two parts so that no wave waits for the first to issue the second:
// (a) the step's counts, its first task's block pairs, the records of the entries it
// subtracts from, read during the step before's sums; (b) those entries, read while
// that step's columns are factored.
constexpr int kStepEntries = (kStepBlks * 36 + kTreeThreads - 1) / kTreeThreads;   // per thread
struct StepHead {   // a record of G.steps, read two steps ahead
  int q0, nq, f0, nf, b0, nb, c0, nc;
};
static_assert(sizeof(StepHead) == 32, "a step's record is eight ints");
struct StepRegs : StepHead {
  int4 blk[kStepEntries], col;   // col: the record of this wave's (first) column
  int ia, ib, c, h0, h1;
};
struct StepVals {
  double v[kStepEntries], hv;
};

// Tasks of a step: per pair of an update chunk four, of 3 x 3 entries of L_rk L_ck^T
// each, and per pair of a forward chunk six, a row of L_ck y_k each.  A thread reads
// three rows of each block once for nine entries: with one entry of all four pairs
// per thread the reads (13.8 kB a chunk through the vector cache against 4.6 kB)
// bound the sums, 4.6 k cycles per 512 tasks; all pairs of a tile in one thread
// need more registers than there are.
constexpr int kUpdTasks = 4 * kPgoChunk, kFwdTasks = 6 * kPgoChunk;   // per chunk

// The block pair of task t of a step (update chunks first, then forward chunks), -1
// past a chunk's end.
__device__ __forceinline__ void step_pair(const PgoDev& G, const StepRegs& R, int t, int& ia, int& ib) {
  const int nu = R.nq * kUpdTasks, u = t - nu;
  const int32_t* p = t < nu ? G.step_ab + 2 * kPgoChunk * ((long long)R.q0 + t / kUpdTasks) + (t >> 2) % kPgoChunk
                            : G.step_bc + 2 * kPgoChunk * ((long long)R.f0 + u / kFwdTasks) + u / 6 % kPgoChunk;
  ia = p[0];
  ib = p[kPgoChunk];
}

__device__ __forceinline__ StepHead step_head(const PgoDev& G, int s) {
  return reinterpret_cast<const StepHead*>(G.steps)[s];
}

__device__ __forceinline__ void step_fetch(const PgoDev& G, const StepHead& H, int wave, StepRegs& R) {
  const int tid = threadIdx.x;
  static_cast<StepHead&>(R) = H;
  R.col = reinterpret_cast<const int4*>(G.step_col)[2 * ((long long)R.c0 + min(wave, R.nc - 1))];
  if (R.nq < 0) return;   // a large column
  const int4* blks = reinterpret_cast<const int4*>(G.step_blk) + R.b0;
#pragma unroll
  for (int k = 0; k < kStepEntries; ++k) {
    const int t = tid + k * kTreeThreads;
    R.blk[k] = blks[t < R.nb * 36 ? t / 36 : 0];
  }
  const int32_t* col = G.step_col + 8 * ((long long)R.c0 + (tid < R.nc * 6 ? tid / 6 : 0));
  R.c = col[0];
  R.h0 = col[4];
  R.h1 = col[5];
  if (tid < R.nq * kUpdTasks + R.nf * kFwdTasks) step_pair(G, R, tid, R.ia, R.ib);
}

__device__ __forceinline__ void step_values(const PgoWork& W, const StepRegs& R, StepVals& V) {
  if (R.nq < 0) return;
#pragma unroll
  for (int k = 0; k < kStepEntries; ++k)
    V.v[k] = W.L[36 * (long long)R.blk[k].x + (threadIdx.x + k * kTreeThreads) % 36];
  V.hv = W.y[6 * R.c + threadIdx.x % 6];
}

// One task of a step into LDS; a pair past its chunk's end counts as zero.
__device__ __forceinline__ void step_task(const PgoWork& W, TreeLds& S, int t, int nu, int ia, int ib) {
  if (t < nu) {
    const int r0 = (t & 2) ? 3 : 0, c0 = (t & 1) ? 3 : 0;
    double la[18], lb[18];
    const double* La = W.L + 36 * (long long)max(ia, 0) + 6 * r0;
    const double* Lb = W.L + 36 * (long long)max(ib, 0) + 6 * c0;
#pragma unroll
    for (int m = 0; m < 18; ++m) {
      la[m] = La[m];
      lb[m] = Lb[m];
    }
    double* out = S.part + 36 * (t >> 2) + 6 * r0 + c0;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double x = 0.0;
#pragma unroll
        for (int m = 0; m < 6; ++m) x += la[6 * r + m] * lb[6 * c + m];
        out[6 * r + c] = ia >= 0 ? x : 0.0;
      }
  } else {
    const int u = t - nu;
    const double* La = W.L + 36 * (long long)max(ia, 0) + 6 * (u % 6);
    const double* yk = W.y + 6 * max(ib, 0);
    double x = 0.0;
#pragma unroll
    for (int m = 0; m < 6; ++m) x += La[m] * yk[m];
    S.fwd[u] = ia >= 0 ? x : 0.0;
  }
}

// v minus the chunks q0 .. q1 - 1 in order, each the sum of its kPgoChunk pairs'
// products in order (pair stride `stride`); four chunks' reads in flight.
__device__ __forceinline__ double minus_chunks(double v, const double* p, int stride, int q0, int q1) {
  for (int q = q0; q < q1; q += 4) {
    double x[4][kPgoChunk];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < kPgoChunk; ++k) x[j][k] = p[stride * (kPgoChunk * min(q + j, q1 - 1) + k)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < kPgoChunk; ++k) acc += x[j][k];
      if (q + j < q1) v -= acc;
    }
  }
  return v;
}

// The steps [s0, s1) of the factorisation.
__device__ __forceinline__ void pgo_tree_factor(const PgoDev& G, const PgoWork& W, int s0, int s1, TreeLds& S) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (s0 >= s1) return;
  StepRegs R, N;
  StepVals V;
  StepHead H = step_head(G, min(s0 + 1, s1 - 1));
  step_fetch(G, step_head(G, s0), wave, R);
  step_values(W, R, V);
  for (int s = s0; s < s1; ++s) {
    if (S.fail) break;
    const int nc = R.nc;
    if (s + 1 < s1) {
      step_fetch(G, H, wave, N);
      H = step_head(G, min(s + 2, s1 - 1));
    }
    if (R.nq < 0) {   // one large column, through memory
      const int c = R.col.x, bd = R.col.y, n = R.col.z;
      pgo_big_sums(G, W, c, bd, n, tid, kTreeThreads);
      __syncthreads();
      pgo_big_subtract(G, W, c, bd, n, tid, kTreeThreads);
      __syncthreads();
      if (s + 1 < s1) step_values(W, N, V);
      // every wave factors the diagonal block and solves its share of the rows in place
      double m[36];
      const bool ok = pgo_rows(W, c, bd, n, W.L + 36 * (long long)bd, W.y + 6 * c, tid, kTreeThreads, &S.fail, m);
      __syncthreads();   // the block has been read by all
      if (ok && tid == 0) pgo_store_diag(W, bd, m);
    } else {
      // (1) the chunks' sums
      const int nu = R.nq * kUpdTasks, nt = nu + R.nf * kFwdTasks;
      if (tid < nt) step_task(W, S, tid, nu, R.ia, R.ib);
      for (int t = tid + kTreeThreads; t < nt; t += kTreeThreads) {
        int ia, ib;
        step_pair(G, R, t, ia, ib);
        step_task(W, S, t, nu, ia, ib);
      }
      __syncthreads();
      // (2) subtracted in chunk order
#pragma unroll
      for (int k = 0; k < kStepEntries; ++k) {
        const int t = tid + k * kTreeThreads;
        if (t < R.nb * 36) S.blk[t] = minus_chunks(V.v[k], S.part + t % 36, 36, R.blk[k].y, R.blk[k].z);
      }
      if (tid < nc * 6) S.rhs[tid] = minus_chunks(V.hv, S.fwd + tid % 6, 6, R.h0, R.h1);
      __syncthreads();
      // (3) one wave per column
      if (s + 1 < s1) step_values(W, N, V);
      for (int i = wave; i < nc; i += kTreeThreads / 64) {
        int4 col = R.col;
        if (i != wave) col = reinterpret_cast<const int4*>(G.step_col)[2 * ((long long)R.c0 + i)];
        double m[36];
        if (pgo_rows(W, col.x, col.y, col.z, S.blk + 36 * col.w, S.rhs + 6 * i, lane, 64, &S.fail, m) && lane == 0)
          pgo_store_diag(W, col.y, m);
      }
    }
    __syncthreads();
    R = N;
  }
}

// What a thread reads of a step of the back substitution that the later steps do not
// change: a block's product row, and (six neighbouring lanes per column, ten columns
// per wave) a column's record, right-hand side and diagonal block.
struct BackRegs {
  int nb, nc, row;
  bool big;
  int c, bd, n, b0;
  double l[6], y, d[21];
};
static_assert(kStepBlks * 6 <= kTreeThreads && kStepCols <= 10 * (kTreeThreads / 64),
              "a step's block rows and columns have a thread each");

__device__ __forceinline__ void back_fetch(const PgoDev& G, const PgoWork& W, int s, BackRegs& R) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* st = G.steps + 8 * (long long)s;
  R.big = st[1] < 0;
  R.nb = st[5];
  R.nc = st[7];
  R.row = -1;
  if (!R.big && tid < R.nb * 6) {
    const int4 b = reinterpret_cast<const int4*>(G.step_blk)[st[4] + tid / 6];
    R.row = b.w;
    const double* L = W.L + 36 * (long long)b.x + tid % 6;
#pragma unroll
    for (int m = 0; m < 6; ++m) R.l[m] = L[6 * m];
  }
  const int i = 10 * wave + lane / 6;
  R.c = -1;
  if (R.big || (lane < 60 && i < R.nc)) {   // (a large column's blocks are every thread's)
    const int32_t* col = G.step_col + 8 * ((long long)st[6] + (R.big ? 0 : i));
    R.bd = col[1];
    R.n = col[2];
    R.b0 = col[3];
    if (lane < 60 && i < R.nc) R.c = col[0];
  }
  if (R.c >= 0) {
    R.y = W.y[6 * R.c + lane % 6];
    const double* D = W.L + 36 * (long long)R.bd;
#pragma unroll
    for (int p = 0, e = 0; p < 6; ++p)
#pragma unroll
      for (int q = 0; q <= p; ++q, ++e) R.d[e] = D[6 * p + q];
  }
}

// The back substitution of the steps [s0, s1), last step first: x_c = L_cc^-T (y_c -
// sum over the column's off-diagonal blocks of L_rc^T x_r).  Every block's product
// row has its own thread; six neighbouring lanes per column subtract them in order,
// exchange the sums and solve the 6x6 triangle, each keeping its own row.
__device__ __forceinline__ void pgo_tree_back(const PgoDev& G, const PgoWork& W, int s0, int s1, TreeLds& S) {
  const int tid = threadIdx.x, a = (tid & 63) % 6;
  if (s0 >= s1) return;
  BackRegs R;
  back_fetch(G, W, s1 - 1, R);
  for (int s = s1 - 1; s >= s0; --s) {
    if (!R.big) {
      if (tid < R.nb * 6) {
        double x = 0.0;
        if (R.row >= 0) {
#pragma unroll
          for (int m = 0; m < 6; ++m) x += R.l[m] * W.x[6 * R.row + m];
        }
        S.blk[tid] = x;
      }
      __syncthreads();
    }
    double v = 0.0;
    if (R.c >= 0) v = R.y;
    if (R.big) {   // as many of the column's product rows at a time as there is room for
      constexpr int kRoom = (int)(sizeof(S.part) / (6 * sizeof(double)));
      for (int k0 = 1; k0 < R.n; k0 += kRoom) {
        const int nk = min(kRoom, R.n - k0);
        for (int t = tid; t < nk * 6; t += kTreeThreads) {
          const int b = R.bd + k0 + t / 6, r = G.blk_row[b];
          const double* L = W.L + 36 * (long long)b + t % 6;
          double x = 0.0;
#pragma unroll
          for (int m = 0; m < 6; ++m) x += L[6 * m] * W.x[6 * r + m];
          S.part[t] = x;
        }
        __syncthreads();
        if (R.c >= 0) v = minus_list(v, S.part + a, 6, nk);
        __syncthreads();
      }
    } else if (R.c >= 0) {
      for (int k = 1; k < R.n; ++k) v -= S.blk[6 * (R.b0 + k) + a];
    }
    S.v[tid] = v;
    __builtin_amdgcn_wave_barrier();   // the six lanes are of one wave, whose LDS operations stay in order
    if (R.c >= 0) {
      double vv[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) vv[q] = S.v[tid - a + q];
#pragma unroll
      for (int k = 5; k >= 0; --k) {
        double t = vv[k];
#pragma unroll
        for (int q = k + 1; q < 6; ++q) t -= R.d[q * (q + 1) / 2 + k] * vv[q];
        vv[k] = t / R.d[k * (k + 1) / 2 + k];
      }
      double mine = vv[0];
#pragma unroll
      for (int q = 1; q < 6; ++q) mine = a == q ? vv[q] : mine;
      W.x[6 * R.c + a] = mine;
    }
    if (s > s0) back_fetch(G, W, s - 1, R);
    __syncthreads();
  }
}

// One tier's groups from g0 on; the last tier is one group, which goes on with the back
// substitution of its own steps and says whether the candidate is valid.
template <bool LAST>
__global__ __launch_bounds__(kTreeThreads) void k_pgo_tree(PgoArgs A, int g0) {
  __shared__ TreeLds S;
  const PgoDev& G = A.G;
  const PgoWork& W = A.W;
  const int g = g0 + blockIdx.x, s0 = G.grp_ptr[g], s1 = G.grp_ptr[g + 1];
  if (threadIdx.x == 0) S.fail = W.istate[4];   // a pivot of an earlier tier
  __syncthreads();
  pgo_tree_factor(G, W, s0, s1, S);
  if (!LAST) return;
  if (S.fail) {
    if (threadIdx.x == 0) {
      W.istate[1] = 0;
      W.istate[3] += 1;
    }
    return;
  }
  pgo_tree_back(G, W, s0, s1, S);
  if (threadIdx.x == 0) W.istate[1] = 1;
}

// The back substitution of one earlier tier's groups.
__global__ __launch_bounds__(kTreeThreads) void k_pgo_back(PgoArgs A, int g0) {
  __shared__ TreeLds S;
  if (A.W.istate[1] == 0) return;
  const int g = g0 + blockIdx.x;
  pgo_tree_back(A.G, A.W, A.G.grp_ptr[g], A.G.grp_ptr[g + 1], S);
}

// Candidate poses Exp(d_i) T_i for the free poses (the others copied); a
// failed factorisation leaves the current poses.
__global__ __launch_bounds__(kPgoEdgeThreads) void k_pgo_candidate(PgoArgs A) {
  const int i = blockIdx.x * kPgoEdgeThreads + threadIdx.x;
  if (i >= A.G.n_poses) return;
  const int c = A.G.col_of_pose[i];
  const double* T = A.poses + 12 * (long long)i;
  double* out = A.W.cand + 12 * (long long)i;
  if (c < 0 || A.W.istate[1] == 0) {
#pragma unroll
    for (int k = 0; k < 12; ++k) out[k] = T[k];
  } else {
    double Dx[12];
    exp_se3(A.W.x + 6 * c, Dx);
    tcompose(Dx, T, out);
  }
}

hipError_t run_pgo(const PgoArgs& A) {
  hipStream_t s = (hipStream_t)A.stream;
  const int eb = (A.G.n_edges + kPgoEdgeThreads - 1) / kPgoEdgeThreads;
  const int ab = (A.G.n_blocks * 6 + A.G.n_free + kPgoEdgeThreads - 1) / kPgoEdgeThreads;
  const int pb = (A.G.n_poses + kPgoEdgeThreads - 1) / kPgoEdgeThreads;
  const int n_it = A.settings.max_iters;
  auto prepare = [&]() {
    // the assembly also clears the pivot-failure flag, so it runs even when
    // there is nothing to gather
    hipLaunchKernelGGL(k_pgo_assemble, dim3(ab > 0 ? ab : 1), dim3(kPgoEdgeThreads), 0, s, A);
    for (int t = 0; t < A.n_tiers; ++t) {
      const int g0 = A.tier_ptr[t], ng = A.tier_ptr[t + 1] - g0;
      if (t + 1 == A.n_tiers) hipLaunchKernelGGL(k_pgo_tree<true>, dim3(ng), dim3(kTreeThreads), 0, s, A, g0);
      else hipLaunchKernelGGL(k_pgo_tree<false>, dim3(ng), dim3(kTreeThreads), 0, s, A, g0);
    }
    for (int t = A.n_tiers - 2; t >= 0; --t) {
      const int g0 = A.tier_ptr[t], ng = A.tier_ptr[t + 1] - g0;
      hipLaunchKernelGGL(k_pgo_back, dim3(ng), dim3(kTreeThreads), 0, s, A, g0);
    }
    hipLaunchKernelGGL(k_pgo_candidate, dim3(pb), dim3(kPgoEdgeThreads), 0, s, A);
  };
  if (eb > 0) hipLaunchKernelGGL(k_pgo_edges, dim3(eb), dim3(kPgoEdgeThreads), 0, s, A, 1);
  hipLaunchKernelGGL(k_pgo_decide, dim3(1), dim3(kPgoStepThreads), 0, s, A, 0, -1, n_it == 0 ? 1 : 0);
  if (n_it > 0) prepare();
  for (int it = 0; it < n_it; ++it) {
    if (eb > 0) hipLaunchKernelGGL(k_pgo_edges, dim3(eb), dim3(kPgoEdgeThreads), 0, s, A, 0);
    hipLaunchKernelGGL(k_pgo_decide, dim3(1), dim3(kPgoStepThreads), 0, s, A, 1, it, it + 1 == n_it ? 1 : 0);
    if (it + 1 < n_it) prepare();
  }
  return hipGetLastError();
}

}  // namespace ba
