// Device geometry and wave-level helpers shared by the window solver
// (kernels.hip) and the motion-only solver (pnp.hip).
//
// Residual and kernel (paper Sec. 2.2, Eq. 2): r = pi(T_cb T_bw p) - o with a
// pinhole pi, the Huber kernel on s = |r|^2; pose updates by the left
// perturbation T <- Exp(xi) T, xi = (rho, phi).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace ba {

// 1/x and 1/sqrt(x) in FP64: the hardware estimates refined by two Newton
// steps each (a few ulp for finite normal x; not correctly rounded).
__device__ __forceinline__ double recip_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  double h = fma(-x * r, r, 1.0);   // r <- r + r (1 - x r^2) / 2
  r = fma(0.5 * r, h, r);
  h = fma(-x * r, r, 1.0);
  return fma(0.5 * r, h, r);
}

// Huber kernel on s = |r|^2: rho, rho', rho''.  delta <= 0 or inf: plain least
// squares.  s == delta^2 takes the inlier branch.
__device__ __forceinline__ void huber(double s, double delta, double& rho, double& d1,
                                      double& d2) {
  if (delta > 0.0 && delta < 1e300 && s > delta * delta) {
    const double ir = rsqrt_nr(s);   // 1 / sqrt(s)
    rho = 2.0 * delta * (s * ir) - delta * delta;
    d1 = delta * ir;
    d2 = -0.5 * delta * ir * ir * ir;
  } else {
    rho = s;
    d1 = 1.0;
    d2 = 0.0;
  }
}

// Linearisation of one observation at (pose R, t | point p).
template <typename Real>
struct Lin {
  double rho_w;     // w * rho(s)
  double d1, d2;    // rho'(s), rho''(s)
  double wo;        // observation weight
  double X, Y, Z;   // camera-frame point
  Real r[2];        // residual pi(x_c) - o
  Real a0[3], a1[3];  // rows of A R_c (A = d pi / d x_c)
  Real xb[3];       // base-frame point
};

template <typename Real>
__device__ __forceinline__ Lin<Real> linearise(const double* __restrict__ xb, const double* C,
                                               double du, double dv, double wo, double delta) {
  Lin<Real> L;
  const double X = C[4] * xb[0] + C[5] * xb[1] + C[6] * xb[2] + C[13];
  const double Y = C[7] * xb[0] + C[8] * xb[1] + C[9] * xb[2] + C[14];
  const double Z = C[10] * xb[0] + C[11] * xb[1] + C[12] * xb[2] + C[15];
  const double iz = recip_nr(Z);
  const double xz = X * iz, yz = Y * iz;
  const double r0 = C[0] * xz - du, r1 = C[1] * yz - dv;
  const double s = r0 * r0 + r1 * r1;
  double rho, d1, d2;
  huber(s, delta, rho, d1, d2);
  L.rho_w = wo * rho;
  L.d1 = d1;
  L.d2 = d2;
  L.wo = wo;
  L.X = X;
  L.Y = Y;
  L.Z = Z;
  L.r[0] = (Real)r0;
  L.r[1] = (Real)r1;
  const double fi = C[0] * iz, gi = C[1] * iz;
  for (int c = 0; c < 3; ++c) {
    L.a0[c] = (Real)(fi * (C[4 + c] - xz * C[10 + c]));
    L.a1[c] = (Real)(gi * (C[7 + c] - yz * C[10 + c]));
    L.xb[c] = (Real)xb[c];
  }
  return L;
}

template <typename Real>
__device__ __forceinline__ void cross3(const Real* a, const Real* b, Real* c) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}

// Lane shift by DPP (row_shr:n within rows of 16 lanes, row_bcast:15 / :31
// across rows) of a 32- or 64-bit value; lanes outside ROWMASK or without a
// source lane read `old`.
template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_i(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWMASK, 0xf, false);
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_r(float x) {
  return __int_as_float(dpp_i<CTRL, ROWMASK>(0, __float_as_int(x)));
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_r(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = dpp_i<CTRL, ROWMASK>(0, (int)(b & 0xffffffffll));
  const int hi = dpp_i<CTRL, ROWMASK>(0, (int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Value of a double in lane `src` (wave-uniform) to every lane, by readlane.
__device__ __forceinline__ double wave_bcast(double x, int src) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Exchange of 64-bit values between lane groups: rows 2-3 of a with rows 0-1
// of b (permlane32), odd rows of a with even rows of b (permlane16).
__device__ __forceinline__ void swap_rows32(double& a, double& b) {
  const long long ia = __double_as_longlong(a), ib = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ia, (unsigned)ib, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ia >> 32), (unsigned)(ib >> 32), false, false);
  a = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
  b = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ void swap_rows16(double& a, double& b) {
  const long long ia = __double_as_longlong(a), ib = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ia, (unsigned)ib, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ia >> 32), (unsigned)(ib >> 32), false, false);
  a = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
  b = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// Sum and maximum over the wave in every lane, as an xor butterfly over lane bits
// 5, 4, 3, 2, 1, 0 adds them: permlane swaps for the rows, then rotations within a
// row (after step 8 the lanes l and l ^ 8 agree, so a rotation by 4 reads the value
// of l ^ 4, and so on).  No LDS, so no bpermute latency per step.
__device__ __forceinline__ double wave_sum(double v) {
  double a = v, b = v;
  swap_rows32(a, b);
  v = a + b;
  a = b = v;
  swap_rows16(a, b);
  v = a + b;
  v += dpp_r<0x128, 0xf>(v);   // row_ror:8
  v += dpp_r<0x124, 0xf>(v);
  v += dpp_r<0x122, 0xf>(v);
  v += dpp_r<0x121, 0xf>(v);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  double a = v, b = v;
  swap_rows32(a, b);
  v = fmax(a, b);
  a = b = v;
  swap_rows16(a, b);
  v = fmax(a, b);
  v = fmax(v, dpp_r<0x128, 0xf>(v));
  v = fmax(v, dpp_r<0x124, 0xf>(v));
  v = fmax(v, dpp_r<0x122, 0xf>(v));
  v = fmax(v, dpp_r<0x121, 0xf>(v));
  return v;
}

// SE(3) exponential of xi = (rho, phi) as a 3x4 [R | t].  The coefficients
// A = sin(th)/th, B = (1 - cos th)/th^2, C = (th - sin th)/th^3 come from
// their power series in th^2 below th = 1 (nine terms: the first omitted one
// is under 1e-17, and the series has no cancellation), and from the closed
// forms above it.
__device__ __forceinline__ void exp_se3(const double* xi, double* T /*3x4*/) {
  const double rx = xi[0], ry = xi[1], rz = xi[2];
  const double px = xi[3], py = xi[4], pz = xi[5];
  const double th2 = px * px + py * py + pz * pz;
  double A, B, Cc;
  if (th2 < 1.0) {
    // A = 1 - t/(2*3) (1 - t/(4*5) (...)), B = (1 - t/(3*4) (...)) / 2,
    // C = (1 - t/(4*5) (...)) / 6, t = th^2
    double a = 1.0, b = 1.0, c = 1.0;
#pragma unroll
    for (int k = 8; k >= 0; --k) {
      const double n = 2.0 * k;
      a = fma(-th2 * (1.0 / ((n + 2.0) * (n + 3.0))), a, 1.0);
      b = fma(-th2 * (1.0 / ((n + 3.0) * (n + 4.0))), b, 1.0);
      c = fma(-th2 * (1.0 / ((n + 4.0) * (n + 5.0))), c, 1.0);
    }
    A = a;
    B = 0.5 * b;
    Cc = c / 6.0;
  } else {
    const double th = sqrt(th2);
    A = sin(th) / th;
    const double s = sin(0.5 * th);
    B = 2.0 * s * s / th2;
    Cc = (th - sin(th)) / (th2 * th);
  }
  const double K[9] = {0, -pz, py, pz, 0, -px, -py, px, 0};
  double K2[9];
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      K2[3 * a + b] = K[3 * a] * K[b] + K[3 * a + 1] * K[3 + b] + K[3 * a + 2] * K[6 + b];
  double R[9], J[9];
  for (int k = 0; k < 9; ++k) {
    const double I = (k % 4 == 0) ? 1.0 : 0.0;
    R[k] = I + A * K[k] + B * K2[k];
    J[k] = I + B * K[k] + Cc * K2[k];
  }
  for (int a = 0; a < 3; ++a) {
    T[4 * a] = R[3 * a];
    T[4 * a + 1] = R[3 * a + 1];
    T[4 * a + 2] = R[3 * a + 2];
    T[4 * a + 3] = J[3 * a] * rx + J[3 * a + 1] * ry + J[3 * a + 2] * rz;
  }
}

// a -= b(s, C) m with b(s, C) the s of lane C of the own row of sixteen lanes: one
// v_fmac_f64 with a row broadcast instead of two lane reads and an fma.  The compiler
// does not see the DPP reads, so the two wait states that they need after a VALU write
// of s lead each block.  Nor does it see the writes: a lane read of a block's output
// needs one instruction in between and a DPP read or lane swap two.  The one such read is
// panel_steps's of the next pivot, which sub_row writes first of two; the wave sums and
// swaps of the kernels that use the blocks read nothing that a block wrote.
#define BA_FMAC_ROW(d, s, m, c) "v_fmac_f64_dpp %" #d ", -%" #s ", %" #m " row_newbcast:%" #c " row_mask:0xf bank_mask:0xf\n"
// one broadcast column over two accumulators: a0 -= b(s, C) m0, a1 -= b(s, C) m1
template <int C>
__device__ __forceinline__ void sub_row(double& a0, double& a1, double s, double m0, double m1) {
  __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 2, 3, 5) BA_FMAC_ROW(1, 2, 4, 5)
                   : "+&v"(a0), "+&v"(a1)
                   : "v"(s), "v"(m0), "v"(m1), "n"(C));
}
template <int C>
__device__ __forceinline__ void sub_row2(double& a0, double& a1, double& b0, double& b1, double s, double m0,
                                         double m1) {
  __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 4, 5, 7) BA_FMAC_ROW(1, 4, 6, 7) BA_FMAC_ROW(2, 4, 5, 8)
                       BA_FMAC_ROW(3, 4, 6, 8)
                   : "+&v"(a0), "+&v"(a1), "+&v"(b0), "+&v"(b1)
                   : "v"(s), "v"(m0), "v"(m1), "n"(C), "n"(C + 1));
}
// columns C .. C + 3 of x and y
template <int C, int N>
__device__ __forceinline__ void sub_row4(double (&x)[N], double (&y)[N], double s, double m0, double m1) {
  __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 8, 9, 11) BA_FMAC_ROW(1, 8, 10, 11) BA_FMAC_ROW(2, 8, 9, 12)
                       BA_FMAC_ROW(3, 8, 10, 12) BA_FMAC_ROW(4, 8, 9, 13) BA_FMAC_ROW(5, 8, 10, 13)
                           BA_FMAC_ROW(6, 8, 9, 14) BA_FMAC_ROW(7, 8, 10, 14)
                   : "+&v"(x[C]), "+&v"(y[C]), "+&v"(x[C + 1]), "+&v"(y[C + 1]), "+&v"(x[C + 2]), "+&v"(y[C + 2]),
                     "+&v"(x[C + 3]), "+&v"(y[C + 3])
                   : "v"(s), "v"(m0), "v"(m1), "n"(C), "n"(C + 1), "n"(C + 2), "n"(C + 3));
}
// columns C .. N - 1 of x and y
template <int C, int N>
__device__ __forceinline__ void sub_rows(double (&x)[N], double (&y)[N], double s, double m0, double m1) {
  if constexpr (C + 3 < N) {
    sub_row4<C, N>(x, y, s, m0, m1);
    sub_rows<C + 4, N>(x, y, s, m0, m1);
  } else if constexpr (C + 1 < N) {
    sub_row2<C>(x[C], y[C], x[C + 1], y[C + 1], s, m0, m1);
    sub_rows<C + 2, N>(x, y, s, m0, m1);
  } else if constexpr (C < N) {
    sub_row<C>(x[C], y[C], s, m0, m1);
  }
}
// a[C] -= b(s, C) m, C = 0 .. 5
__device__ __forceinline__ void sub_vec6(double (&a)[6], double s, double m) {
  __asm__ volatile("s_nop 1\n" BA_FMAC_ROW(0, 6, 7, 8) BA_FMAC_ROW(1, 6, 7, 9) BA_FMAC_ROW(2, 6, 7, 10)
                       BA_FMAC_ROW(3, 6, 7, 11) BA_FMAC_ROW(4, 6, 7, 12) BA_FMAC_ROW(5, 6, 7, 13)
                   : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3]), "+&v"(a[4]), "+&v"(a[5])
                   : "v"(s), "v"(m), "n"(0), "n"(1), "n"(2), "n"(3), "n"(4), "n"(5));
}

__device__ __forceinline__ void pin(double& v) { __asm__ volatile("" : "+v"(v)); }   // not moved past a block above

// Step J of a Cholesky factorisation of N columns in panels: each row of sixteen lanes
// holds in w the N entries of the block's rows (lanes 0 to N - 1: row r, its column r
// being the pivot's) and of columns to solve (the other lanes), in p more columns.
// Column J of the panels is scaled by the pivot's reciprocal root ir (which takes the
// pivot's place), then subtracted from the later columns, right-looking, and its
// products with p's rows 0 to N - 1 from the next block's sums aw (w's lanes) and ap
// (p's).  The next pivot's root (an estimate and one third-order refinement, as rsqrt
// takes it) is worked out between the products.  A pivot past the first that is not
// positive and finite makes it NaN and with it every later pivot; the last root is returned.
template <int J, int N>
__device__ __forceinline__ double panel_steps(double (&w)[N], double (&p)[N], double (&aw)[N], double (&ap)[N],
                                              int row, double ir) {
  w[J] = row == J ? ir : w[J] * ir;
  p[J] *= ir;
  if constexpr (J < N - 1) {
    constexpr int H = N > 8 ? 4 : 0;   // products before the estimate's first refinement step
    sub_row<J + 1>(w[J + 1], p[J + 1], w[J], w[J], p[J]);
    const double d = wave_bcast(w[J + 1], J + 1);
    double y = __builtin_amdgcn_rsq(d);
    pin(y);
    if constexpr (H > 0) sub_row4<0, N>(aw, ap, p[J], w[J], p[J]);
    double t = y * -d;
    pin(t);
    sub_row<H>(aw[H], ap[H], p[J], w[J], p[J]);
    double e = fma(t, y, 1.0);
    pin(e);
    sub_row4<H + 1, N>(aw, ap, p[J], w[J], p[J]);
    double m = y * e;
    pin(m);
    double q = fma(e, 0.375, 0.5);
    pin(q);
    sub_rows<H + 5, N>(aw, ap, p[J], w[J], p[J]);
    double in = fma(m, q, y);
    pin(in);
    sub_rows<J + 2, N>(w, p, w[J], w[J], p[J]);
    return panel_steps<J + 1, N>(w, p, aw, ap, row, in);
  } else {
    sub_rows<0, N>(aw, ap, p[J], w[J], p[J]);
    return ir;
  }
}

// All N steps; false when a pivot is not positive and finite (the same in every lane).
// The first root is tested too: an infinite first pivot's is 0, and the columns that it
// scales to zero leave the later pivots finite.
template <int N>
__device__ __forceinline__ bool factor_panels(double (&w)[N], double (&p)[N], double (&aw)[N], double (&ap)[N],
                                              int row) {
  const double first = rsqrt(wave_bcast(w[0], 0));
  const double last = panel_steps<0, N>(w, p, aw, ap, row, first);
  return first > 0.0 && last > 0.0 && isfinite(last);
}

}  // namespace ba
