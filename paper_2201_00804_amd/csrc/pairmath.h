// Per-pair arithmetic of the real-space kernels: radial coefficients of the
// screened, damped and bare kernels and the multipole contractions written
// out in closed form.
//
// Radial coefficients c_n(r) (c_{n+1} = -c_n'/r) define every interaction
// tensor.  Kernels:
//   bare     c0_n = (2n-1)!! / r^(2n+1)
//   Ewald    B_0 = erfc(beta r)/r,
//            B_n = ((2n-1) B_{n-1} + (2 beta^2)^n exp(-beta^2 r^2)/(beta sqrt(pi))) / r^2
//   Thole    damped c_n = lambda_{2n+1} c0_n with 1 - lambda_{2n+1} = P_n(x) exp(-x),
//            x = a r^3 s_i s_j, s = abar^-1/2, and
//            P_1 = 1, P_2 = 1 + x, P_3 = 1 + x + 3x^2/5,
//            P_4 = 1 + x + 18x^2/35 + 9x^3/35
//            (each from the previous by P_{n+1} = P_n + 3x/(2n+1) (P_n - P_n'),
//            which makes each damped tensor the derivative of the one below).
// Class coefficients with E_n the base kernel (B_n periodic, c0_n cluster):
//   excluded pair (same molecule, permanent involved):  c_n = E_n - c0_n
//   damped pair  (polarizable-polarizable):              c_n = E_n - P_n e^-x c0_n
//   plain pair:                                          c_n = E_n
//
// Multipole convention: the potential of site j at R = r - r_j is
// [q_j - d_j.grad + 1/3 Theta_j:grad grad] G(R) and the energy of site i in a
// potential phi is [q_i + d_i.grad + 1/3 Theta_i:grad grad] phi at r_i, with
// Theta the traceless Buckingham quadrupole.  Expanding with
// grad^n G in terms of deltas, R and c_n gives U = sum_n c_n P_n with
//   P0 = qi qj
//   P1 = qi (dj.R) - qj (di.R) + di.dj
//   P2 = (qi R.Tj.R + qj R.Ti.R)/3 - (di.R)(dj.R) + 2/3 (di.Tj.R - dj.Ti.R)
//        + 2/9 Ti:Tj
//   P3 = ((dj.R)(R.Ti.R) - (di.R)(R.Tj.R))/3 - 4/9 (Ti.R).(Tj.R)
//   P4 = (R.Ti.R)(R.Tj.R)/9
// and the force on i, F = -dU/dR = R sum_n c_{n+1} P_n - sum_n c_n grad P_n.
#pragma once
#include "common.h"
#include "erfcx_fit.h"

namespace sibfa {

// erfcx(x) = exp(x^2) erfc(x) for x >= 0: the Chebyshev series of
// erfcx_fit.h in t = 1 / (1 + p x), x clamped to kErfcxMax (past it erfc is
// below 2e-17).  The Ewald recursion multiplies by the exp(-x^2) it needs
// anyway, so erfc costs a reciprocal and a short series.  Relative error
// about 1e-14 (FP64) and 7e-7 (FP32).
template <typename R>
__device__ __forceinline__ R dev_erfcx(R x);
template <>
__device__ __forceinline__ double dev_erfcx<double>(double x) {
  x = fmin(x, kErfcxMax);
  const double d = 1.0 + kErfcxPF64 * x;
  // single-precision reciprocal, then two Newton steps (1e-7 -> 1e-14 -> exact)
  double t = (double)__builtin_amdgcn_rcpf((float)d);
  t = t * fma(-d, t, 2.0);
  t = t * fma(-d, t, 2.0);
  const double u = fma(t - kErfcxT0F64, 2.0 / (1.0 - kErfcxT0F64), -1.0);
  const double u2 = 2.0 * u;
  double b1 = 0.0, b2 = 0.0;
#pragma unroll
  for (int k = kErfcxDegF64; k >= 1; --k) {
    const double b = fma(u2, b1, kErfcxCF64[k] - b2);
    b2 = b1;
    b1 = b;
  }
  return fma(u, b1, kErfcxCF64[0] - b2);
}
template <>
__device__ __forceinline__ float dev_erfcx<float>(float x) {
  x = fminf(x, (float)kErfcxMax);
  const float t = __builtin_amdgcn_rcpf(1.0f + kErfcxPF32 * x);
  const float u = fmaf(t - kErfcxT0F32, 2.0f / (1.0f - kErfcxT0F32), -1.0f);
  const float u2 = 2.0f * u;
  float b1 = 0.0f, b2 = 0.0f;
#pragma unroll
  for (int k = kErfcxDegF32; k >= 1; --k) {
    const float b = fmaf(u2, b1, kErfcxCF32[k] - b2);
    b2 = b1;
    b1 = b;
  }
  return fmaf(u, b1, kErfcxCF32[0] - b2);
}

template <typename R>
__device__ __forceinline__ R dev_exp(R x);
template <>
__device__ __forceinline__ double dev_exp<double>(double x) { return exp(x); }
// FP32: the hardware 2^x (1 ulp) of x log2(e); the rounding of the product
// adds a relative error of at most 2^-24 |x log2 e| (8e-7 at the Ewald
// recursion's largest argument, 13), within the FP32 path's own rounding.
// The arguments here are never positive; below -126 / log2(e) the result
// flushes to zero, as the true values are then under FP32's normal range.
template <>
__device__ __forceinline__ float dev_exp<float>(float x) {
  return __builtin_amdgcn_exp2f(x * 1.44269504088896341f);
}

template <typename R>
__device__ __forceinline__ R dev_rsqrt(R x);
template <>
__device__ __forceinline__ double dev_rsqrt<double>(double x) { return rsqrt(x); }
template <>
__device__ __forceinline__ float dev_rsqrt<float>(float x) { return rsqrtf(x); }

// bare c0_0..c0_N
template <typename R, int N>
__device__ __forceinline__ void bare_coeffs(R rinv, R rinv2, R c[N + 1]) {
  c[0] = rinv;
#pragma unroll
  for (int n = 1; n <= N; ++n) c[n] = R(2 * n - 1) * c[n - 1] * rinv2;
}

// Ewald real-space B_0..B_N
template <typename R, int N>
__device__ __forceinline__ void ewald_coeffs(R r, R rinv, R rinv2, R beta, R B[N + 1]) {
  const R br = beta * r;
  const R ex = dev_exp<R>(-br * br);
  const R g = ex * (R(1) / (beta * R(kSqrtPi)));
  B[0] = ex * dev_erfcx<R>(br) * rinv;
  const R t = R(2) * beta * beta;
  R tn = t;
#pragma unroll
  for (int n = 1; n <= N; ++n) {
    B[n] = (R(2 * n - 1) * B[n - 1] + tn * g) * rinv2;
    tn *= t;
  }
}

// 1 - lambda_{2n+1} = P_n(x) e^-x, n = 1..4 (tp[0] unused, set 0)
template <typename R>
__device__ __forceinline__ void thole_tp(R x, R tp[5]) {
  const R e = dev_exp<R>(-x);
  const R x2 = x * x;
  tp[0] = R(0);
  tp[1] = e;
  tp[2] = (R(1) + x) * e;
  tp[3] = (R(1) + x + R(0.6) * x2) * e;
  tp[4] = (R(1) + x + R(18.0 / 35.0) * x2 + R(9.0 / 35.0) * x2 * x) * e;
}

// The same in FP64 for the kernels that evaluate every pair of a list
// (200 to 300 FP64 instructions each, which is what bounds them): 2^k times a
// polynomial of degree 11 for exp(-x^2), without the library's special cases
// (the argument is finite and never positive; below -700 it is taken there,
// 1e-304), and the erfcx series by Horner's rule, half Clenshaw's steps.
// a b + c with the constant c in scalar registers: the compiler's own choice,
// an add into a copy of c, keeps some 40 constants in 80 vector registers
// over the pair loops: 256 registers, and one wavefront per SIMD, in the
// force kernel.
__device__ __forceinline__ double fma_const(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}
__device__ __forceinline__ double exp_neg(double x) {
  x = fmax(x, -700.0);
  const double k = rint(x * 1.4426950408889634);
  const double r = fma(k, -2.3190468138462996e-17, fma(k, -0.6931471805599453, x));
  double q = kExpQ[kExpDeg];
#pragma unroll
  for (int m = kExpDeg - 1; m >= 0; --m) q = fma_const(q, r, kExpQ[m]);
  return ldexp(fma(r * r, q, r) + 1.0, (int)k);
}

// 1 / sqrt(x): the hardware's estimate and one third-order step.
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

__device__ __forceinline__ double erfcx_horner(double x) {
  x = fmin(x, kErfcxMax);
  const double d = fma(kErfcxPF64, x, 1.0);
  double t = (double)__builtin_amdgcn_rcpf((float)d);
  t = t * fma(-d, t, 2.0);
  t = t * fma(-d, t, 2.0);
  const double u = fma(t - kErfcxT0F64, 2.0 / (1.0 - kErfcxT0F64), -1.0);
  double b = kErfcxMF64[kErfcxDegF64];
#pragma unroll
  for (int k = kErfcxDegF64 - 1; k >= 0; --k) b = fma_const(b, u, kErfcxMF64[k]);
  return b;
}

template <int N>
__device__ __forceinline__ void ewald_coeffs_f64(double r, double rinv, double rinv2, double beta,
                                                 double B[N + 1]) {
  const double br = beta * r;
  const double ex = exp_neg(-br * br);
  B[0] = ex * erfcx_horner(br) * rinv;
  const double t = 2.0 * beta * beta;
  double h = ex * (t / (beta * kSqrtPi));
#pragma unroll
  for (int n = 1; n <= N; ++n) {
    B[n] = fma(double(2 * n - 1), B[n - 1], h) * rinv2;
    h *= t;
  }
}

__device__ __forceinline__ void thole_tp_f64(double x, double tp[5]) {
  const double e = exp_neg(-x);
  tp[0] = 0.0;
  tp[1] = e;
  tp[2] = (1.0 + x) * e;
  tp[3] = fma(x, fma(0.6, x, 1.0), 1.0) * e;
  tp[4] = fma(x, fma(x, fma(9.0 / 35.0, x, 18.0 / 35.0), 1.0), 1.0) * e;
}

template <typename R>
struct MP {
  R q;
  R d[3];
  R t[6];   // xx, xy, xz, yy, yz, zz
};

template <typename R>
__device__ __forceinline__ void tvec(const R t[6], const R v[3], R o[3]) {
  o[0] = t[0] * v[0] + t[1] * v[1] + t[2] * v[2];
  o[1] = t[1] * v[0] + t[3] * v[1] + t[4] * v[2];
  o[2] = t[2] * v[0] + t[4] * v[1] + t[5] * v[2];
}

// Energy U and force on i (F = -dU/dR) of multipoles A at r_i and B at
// r_j, R = r_i - r_j, with coefficients c[0..5] (c[5] used by the force).
template <typename R, bool WANT_U, bool WANT_F>
__device__ __forceinline__ void mp_pair(const R c[6], const MP<R>& A, const MP<R>& B,
                                        const R Rv[3], R& U, R F[3]) {
  const R dri = A.d[0] * Rv[0] + A.d[1] * Rv[1] + A.d[2] * Rv[2];
  const R drj = B.d[0] * Rv[0] + B.d[1] * Rv[1] + B.d[2] * Rv[2];
  const R dij = A.d[0] * B.d[0] + A.d[1] * B.d[1] + A.d[2] * B.d[2];
  R qir[3], qjr[3];
  tvec(A.t, Rv, qir);
  tvec(B.t, Rv, qjr);
  const R qrri = qir[0] * Rv[0] + qir[1] * Rv[1] + qir[2] * Rv[2];
  const R qrrj = qjr[0] * Rv[0] + qjr[1] * Rv[1] + qjr[2] * Rv[2];
  const R diqjr = A.d[0] * qjr[0] + A.d[1] * qjr[1] + A.d[2] * qjr[2];
  const R djqir = B.d[0] * qir[0] + B.d[1] * qir[1] + B.d[2] * qir[2];
  const R qq = qir[0] * qjr[0] + qir[1] * qjr[1] + qir[2] * qjr[2];
  const R tt = A.t[0] * B.t[0] + A.t[3] * B.t[3] + A.t[5] * B.t[5] +
               R(2) * (A.t[1] * B.t[1] + A.t[2] * B.t[2] + A.t[4] * B.t[4]);
  const R third = R(1.0 / 3.0);
  const R P0 = A.q * B.q;
  const R P1 = A.q * drj - B.q * dri + dij;
  const R P2 = third * (A.q * qrrj + B.q * qrri) - dri * drj + R(2.0 / 3.0) * (diqjr - djqir) +
               R(2.0 / 9.0) * tt;
  const R P3 = third * (drj * qrri - dri * qrrj) - R(4.0 / 9.0) * qq;
  const R P4 = R(1.0 / 9.0) * qrri * qrrj;
  if (WANT_U) U = c[0] * P0 + c[1] * P1 + c[2] * P2 + c[3] * P3 + c[4] * P4;
  if (WANT_F) {
    const R rad = c[1] * P0 + c[2] * P1 + c[3] * P2 + c[4] * P3 + c[5] * P4;
    R tjdi[3], tidj[3], tiqjr[3], tjqir[3];
    tvec(B.t, A.d, tjdi);
    tvec(A.t, B.d, tidj);
    tvec(A.t, qjr, tiqjr);
    tvec(B.t, qir, tjqir);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const R g1 = A.q * B.d[a] - B.q * A.d[a];
      const R g2 = R(2.0 / 3.0) * (A.q * qjr[a] + B.q * qir[a]) - A.d[a] * drj - B.d[a] * dri +
                   R(2.0 / 3.0) * (tjdi[a] - tidj[a]);
      const R g3 = third * (B.d[a] * qrri - A.d[a] * qrrj) +
                   R(2.0 / 3.0) * (drj * qir[a] - dri * qjr[a]) -
                   R(4.0 / 9.0) * (tiqjr[a] + tjqir[a]);
      const R g4 = R(2.0 / 9.0) * (qir[a] * qrrj + qjr[a] * qrri);
      F[a] = Rv[a] * rad - (c[1] * g1 + c[2] * g2 + c[3] * g3 + c[4] * g4);
    }
  }
}

// Field at r_i of the multipoles B at r_j, R = r_i - r_j, coefficients c[1..3].
template <typename R>
__device__ __forceinline__ void mp_field(const R c[6], const MP<R>& B, const R Rv[3], R E[3]) {
  const R drj = B.d[0] * Rv[0] + B.d[1] * Rv[1] + B.d[2] * Rv[2];
  R qjr[3];
  tvec(B.t, Rv, qjr);
  const R qrrj = qjr[0] * Rv[0] + qjr[1] * Rv[1] + qjr[2] * Rv[2];
  const R rad = B.q * c[1] + drj * c[2] + R(1.0 / 3.0) * qrrj * c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) E[a] = Rv[a] * rad - (B.d[a] * c[1] + R(2.0 / 3.0) * qjr[a] * c[2]);
}

// Derivatives at r_i of the potential phi of multipoles at r_j, summed over
// j: a site's multipoles meet the sums once instead of every pair.  With
// S_k = q c_k + (d.R) c_{k+1} + 1/3 (R Theta R) c_{k+2} and
// W_k = d c_k + 2/3 (Theta R) c_{k+1}, dS_k/dR_a = -R_a S_{k+1} + W_{k+1,a}, so
//   phi            = S_0
//   d_a phi        = -R_a S_1 + W_1a
//   d_a d_b phi    = R_a y_b + R_b y_a + 2/3 c_2 Theta_ab - delta_ab S_1,
//                    y = R S_2 / 2 - W_2
//   d_a d_b d_c phi = -(R_a u_bc + R_b u_ac + R_c u_ab) + delta_ab z_c + delta_ac z_b
//                    + delta_bc z_a,  u_bc = R_b v_c + R_c v_b + 2/3 c_3 Theta_bc,
//                    v = R S_3 / 6 - W_3 / 2,  z = R S_2 - W_2.
// Site i's quadrupole is contracted over b, c with the terms in delta_bc left
// out, as in mp_pair (they meet its trace, which is zero).  The FP64 pair loops
// are bound by their instructions: sums instead of pair energies and forces,
// with the functions above, take 388 vector instructions per entry of the
// force to 270 and 254 of the permanent field to 211; over 160,000 sites
// (cutoff 9, 509 entries each) 1270 us became 810 and 950 became 610.
struct PotSums {
  double e[3];         // d_a phi
  double g[6], s1;     // the second derivatives without their S_1; S_1
  double z[3], k[10];  // z; R_a u_bc + ...: xxx yyy zzz (a third of them), xxy xxz yyx yyz zzx zzy, xyz
};

// A source's S_1..S_3, W_1..W_3 and, of its quadrupole, 2/3 c_2 and 2/3 c_3.
struct PotTerms {
  double S1, S2, S3, W1[3], W2[3], W3[3], k2, k3;
};

// R_a y_b + R_b y_a + k Theta_ab
__device__ __forceinline__ void sym_add(const double R[3], const double y[3], double k,
                                        const double t[6], double g[6]) {
  g[0] = fma(2.0 * R[0], y[0], fma(k, t[0], g[0]));
  g[1] = fma(R[0], y[1], fma(R[1], y[0], fma(k, t[1], g[1])));
  g[2] = fma(R[0], y[2], fma(R[2], y[0], fma(k, t[2], g[2])));
  g[3] = fma(2.0 * R[1], y[1], fma(k, t[3], g[3]));
  g[4] = fma(R[1], y[2], fma(R[2], y[1], fma(k, t[4], g[4])));
  g[5] = fma(2.0 * R[2], y[2], fma(k, t[5], g[5]));
}

// Terms of the first two (TOP 2) or three derivatives' sums; m = d.R,
// t = Theta R, n = R Theta R / 3.
template <int TOP>
__device__ __forceinline__ void pot_terms(const double c[6], const MP<double>& M, double m,
                                          const double t[3], double n, PotTerms& T) {
  T.k2 = (2.0 / 3.0) * c[2];
  T.k3 = (2.0 / 3.0) * c[3];
  T.S1 = fma(n, c[3], fma(m, c[2], M.q * c[1]));
  T.S2 = fma(n, c[4], fma(m, c[3], M.q * c[2]));
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    T.W1[a] = fma(c[1], M.d[a], T.k2 * t[a]);
    T.W2[a] = fma(c[2], M.d[a], T.k3 * t[a]);
  }
  if (TOP == 3) {
    const double k4 = (2.0 / 3.0) * c[4];
    T.S3 = fma(n, c[5], fma(m, c[4], M.q * c[3]));
#pragma unroll
    for (int a = 0; a < 3; ++a) T.W3[a] = fma(c[3], M.d[a], k4 * t[a]);
  }
}

template <int TOP>
__device__ __forceinline__ void pot_add(const PotTerms& T, const double Th[6], const double R[3],
                                        PotSums& P) {
  const double h = 0.5 * T.S2;
  double y[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    P.e[a] += fma(-T.S1, R[a], T.W1[a]);
    y[a] = fma(h, R[a], -T.W2[a]);
    if (TOP == 3) P.z[a] += fma(h, R[a], y[a]);
  }
  sym_add(R, y, T.k2, Th, P.g);
  if (TOP == 3) {
    P.s1 += T.S1;
    const double s6 = (1.0 / 6.0) * T.S3;
    double v[3], u[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = fma(s6, R[a], -0.5 * T.W3[a]);
    sym_add(R, v, T.k3, Th, u);
    const double R2[3] = {2.0 * R[0], 2.0 * R[1], 2.0 * R[2]};
    P.k[0] = fma(R[0], u[0], P.k[0]);
    P.k[1] = fma(R[1], u[3], P.k[1]);
    P.k[2] = fma(R[2], u[5], P.k[2]);
    P.k[3] = fma(R2[0], u[1], fma(R[1], u[0], P.k[3]));
    P.k[4] = fma(R2[0], u[2], fma(R[2], u[0], P.k[4]));
    P.k[5] = fma(R2[1], u[1], fma(R[0], u[3], P.k[5]));
    P.k[6] = fma(R2[1], u[4], fma(R[2], u[3], P.k[6]));
    P.k[7] = fma(R2[2], u[2], fma(R[0], u[5], P.k[7]));
    P.k[8] = fma(R2[2], u[4], fma(R[1], u[5], P.k[8]));
    P.k[9] = fma(R[0], u[4], fma(R[1], u[2], fma(R[2], u[1], P.k[9])));
  }
}

// Energy of multipoles A in the summed potential phi.
__device__ __forceinline__ double pot_energy(const MP<double>& A, double phi, const PotSums& P) {
  const double tg = A.t[0] * P.g[0] + A.t[3] * P.g[3] + A.t[5] * P.g[5] +
                    2.0 * (A.t[1] * P.g[1] + A.t[2] * P.g[2] + A.t[4] * P.g[4]);
  return A.q * phi + (A.d[0] * P.e[0] + A.d[1] * P.e[1] + A.d[2] * P.e[2]) + (1.0 / 3.0) * tg;
}

// Force on multipoles A in the summed potential.
__device__ __forceinline__ void pot_force(const MP<double>& A, const PotSums& P, double F[3]) {
  double dg[3], tz[3];
  tvec(P.g, A.d, dg);
  tvec(A.t, P.z, tz);
  const double tk[3] = {
      3.0 * A.t[0] * P.k[0] + A.t[3] * P.k[5] + A.t[5] * P.k[7] +
          2.0 * (A.t[1] * P.k[3] + A.t[2] * P.k[4] + A.t[4] * P.k[9]),
      A.t[0] * P.k[3] + 3.0 * A.t[3] * P.k[1] + A.t[5] * P.k[8] +
          2.0 * (A.t[1] * P.k[5] + A.t[2] * P.k[9] + A.t[4] * P.k[6]),
      A.t[0] * P.k[4] + A.t[3] * P.k[6] + 3.0 * A.t[5] * P.k[2] +
          2.0 * (A.t[1] * P.k[9] + A.t[2] * P.k[7] + A.t[4] * P.k[8])};
#pragma unroll
  for (int a = 0; a < 3; ++a)
    F[a] += -A.q * P.e[a] - dg[a] + P.s1 * A.d[a] + (1.0 / 3.0) * tk[a] - (2.0 / 3.0) * tz[a];
}

// Field at r_i of a point dipole p at r_j (coefficients c1, c2).
template <typename R>
__device__ __forceinline__ void dip_field(R c1, R c2, const R p[3], const R Rv[3], R E[3]) {
  const R rp = Rv[0] * p[0] + Rv[1] * p[1] + Rv[2] * p[2];
#pragma unroll
  for (int a = 0; a < 3; ++a) E[a] = c2 * rp * Rv[a] - c1 * p[a];
}

}  // namespace sibfa
