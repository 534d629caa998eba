// Batched gas-phase clusters: for every cluster the permanent field and
// E_elec, a block-Jacobi PCG for T mu = E (Eq. 18), E_pol = -1/2 mu.E
// (Eq. 19) and the forces, by direct sums (no cutoff, no neighbour list).
// Forces go through the combined-density identity of the periodic force
// kernel with the bare kernel.
//
// A cluster is small (at most kClSmall sites) or large, by its own size:
//
//   small: one workgroup does everything, records and pair coefficients in
//          LDS (k_cl_small, or beside the large solves: small_apart);
//   large: k_cl_prep  (site records, polarizable compaction),
//          k_cl_field (16 sites per workgroup and step: field and E_elec;
//                      other workgroups of the launch fill the table of
//                      pair coefficients),
//          k_cl_solve (the whole PCG in one workgroup of 768 threads),
//          k_cl_force (16 sites per workgroup and step).
//
// Sixteen lanes share a site in every pair sum, and every reduction runs in
// a fixed order inside one workgroup, so a cluster's results are bitwise
// independent of which other clusters share the batch, of the number of
// workgroups and of whether its coefficients come from the table.
//
// Pair coefficients of a cluster (bare kernel c0_n = (2n-1)!!/r^(2n+1)):
//   different molecules: MM c0; Mmu and mumu (both sites polarizable)
//                        c0 - P_n e^-x c0 (Thole); same molecule: mumu only,
//                        damped; MM and Mmu excluded.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/sibfa_pol.h"
#include "common.h"
#include "pairmath.h"

namespace sibfa {

constexpr int kClBlock = 256;       // threads of every kernel but the large solve
constexpr int kClSolveBlock = 768;
constexpr int kClG = 16;            // lanes per site
constexpr int kClTile = kClBlock / kClG;   // sites per workgroup and step
constexpr int kClMaxSites = SIBFA_BATCH_MAX_SITES;
constexpr int kClMaxPol = SIBFA_BATCH_MAX_POLARIZABLE;
// Small clusters: with 64 sites one workgroup's field and force sums are 16
// steps of 16 sites, about the four launches they save; the coefficient
// table in LDS holds 40 polarizable sites (25 KB; more are re-evaluated).
constexpr int kClSmall = 64;
constexpr int kClSmallTable = 40;
// Do a batch's small clusters run in k_cl_small, before the large ones, or
// beside the large solves?  A solve's workgroup has all registers of a CU, so
// one cluster per CU at a time there and a small one takes a third longer (its
// registers spill); k_cl_small takes two per CU but then the solves wait.  ns
// small and nl large clusters, cs and cl the sums of their costs (cluster_cost)
// and ml the largest: 256 CUs, and half a small cluster for the last round.
// Calls beside / apart (FP64): 1,000 of 2 to 8 waters and one of 64 380 / 431 us,
// and one of 13 359 / 311; 3,000 and one of 64 860 / 704; 200 of 8 to 12 waters
// and 200 of 13 308 / 276; 1,000 of those and 4 of 128 691 / 861.
struct BatchCost {
  int ns, nl, cs, cl, ml;
};
// microseconds of a cluster of n sites, roughly
__host__ __device__ inline int cluster_cost(int n) {
  return n <= kClSmall ? 25 + n : 40 + n / 2;
}
__host__ __device__ inline bool small_apart(const BatchCost& b) {
  constexpr int kCUs = 256;
  if (b.nl == 0 || b.ns == 0) return b.nl == 0;
  if (b.ns + b.nl <= kCUs) return false;
  const int each = b.cs / b.ns, mean = (b.cl + b.cs / 3 * 4) / kCUs + each * 2 / 3;
  const int beside = mean > b.ml ? mean : b.ml;
  const int solves = b.cl / kCUs > b.ml ? b.cl / kCUs : b.ml;
  const int first = b.cs / (2 * kCUs) > each ? b.cs / (2 * kCUs) : each;
  return solves + first < beside;
}
static_assert(kClMaxPol <= kClSolveBlock, "one thread per polarizable site of the large solve");
static_assert(kClSmall <= kClBlock, "one thread per site of a small cluster");

struct ClusterArgs {
  int nclusters;
  int nsites;           // sites in the caller arrays (and scratch capacity)
  const int* off;       // [nclusters + 1] site offsets into the caller arrays
  const int* warm;      // [nclusters] 1: start from mu, or nullptr
  // clusters the large kernels are launched for, -1 after the last
  const int* large;
  // where k_cl_prep writes that list and whether the small clusters run apart,
  // if the host does not know the sizes, or nullptr
  int* list;
  int* apart;
  // start of each cluster's coefficient table in pairs, or -1 (nullptr: no
  // cluster has one)
  const long long* coef_off;
  double2* coef;        // FP64 tables, [np][np] per cluster
  float2* coef32;       // FP32 tables (mixed precision)
  const double* xyz;    // caller arrays, concatenated clusters
  const int* mol;
  const double* q;
  const double* dip;
  const double* quad;
  const double* alpha;
  const double* thole;  // [n] or nullptr (uniform thole_a)
  double thole_a;
  double tol;
  int max_iter;
  // scratch of the large clusters, indexed by global site; polarizable
  // entries are compacted to the front of each cluster's segment
  int* npol;            // [nclusters]
  int* polsite;         // [n] polarizable rank -> site of the cluster
  int* prank;           // [n] site -> polarizable rank, or -1
  double4* rec;         // [n][4] site records (see load_rec)
  double4* E0;          // [n] by polarizable rank
  double* usite;        // [n] MM energy of each site
  // outputs
  double* mu;           // [n][3]
  double* forces;       // [n][3] or nullptr
  double* e_pol;        // [nclusters]
  double* e_elec;
  int* iters;
  double* rms;
  int* status;
};

// ---------------------------------------------------------------- helpers

// Cluster c's site range [base, base + n) from the offsets, and whether it
// is a valid one: 1..kClMaxSites sites inside the nsites of the arrays.
// Offsets validated on the host always pass; offsets that the caller
// keeps on the device are checked here, and a cluster whose range fails
// is reported (E_ARG) without touching its rows.
__device__ __forceinline__ bool cluster_range(const ClusterArgs& a, int c, int& base, int& n) {
  base = a.off[c];
  const int end = a.off[c + 1];
  n = base >= 0 && end > base ? end - base : 0;   // no overflow: both are >= 0
  return n >= 1 && n <= kClMaxSites && end <= a.nsites;
}

// The k-th of count entries of the list of large clusters, -1 past the last.
__device__ __forceinline__ int cluster_at(const ClusterArgs& a, int k, int count) {
  return k < count ? a.large[k] : -1;
}
__device__ __forceinline__ bool large_cluster(const ClusterArgs& a, int c, int& base, int& n) {
  return cluster_range(a, c, base, n) && n > kClSmall;
}

// Sums of one or two values over the NT threads of a block, returned to
// every thread in the same fixed order.  All threads must call it.
template <int NT>
struct BlockSum {
  double* sh;   // [2][NT / 64] in LDS
  __device__ void operator()(double& a, double& b) const {
    constexpr int W = NT / 64;
    a = wave_sum(a);
    b = wave_sum(b);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) {
      sh[w] = a;
      sh[W + w] = b;
    }
    __syncthreads();
    a = b = 0.0;
#pragma unroll 4
    for (int k = 0; k < W; ++k) {
      a += sh[k];
      b += sh[W + k];
    }
  }
  __device__ void operator()(double& a) const {
    double b = 0.0;
    (*this)(a, b);
  }
};

// Site record, four double4: x y z q | d, s = abar^-1/2 (0: not
// polarizable) | Theta xx xy xz yy | Theta yz zz, Thole factor, molecule
// (an integer in the low word).
template <typename R>
struct Site {
  double x[3];
  MP<R> M;
  double s, th;
  int mol;
};

template <typename R>
__device__ __forceinline__ void load_rec(const double4* rec, int i, Site<R>& S) {
  const double4 a = rec[4 * i], b = rec[4 * i + 1], c = rec[4 * i + 2], d = rec[4 * i + 3];
  S.x[0] = a.x; S.x[1] = a.y; S.x[2] = a.z;
  S.M.q = (R)a.w;
  S.M.d[0] = (R)b.x; S.M.d[1] = (R)b.y; S.M.d[2] = (R)b.z;
  S.s = b.w;
  S.M.t[0] = (R)c.x; S.M.t[1] = (R)c.y; S.M.t[2] = (R)c.z; S.M.t[3] = (R)c.w;
  S.M.t[4] = (R)d.x; S.M.t[5] = (R)d.y;
  S.th = d.z;
  S.mol = __double2loint(d.w);
}

__device__ __forceinline__ void store_rec(const ClusterArgs& a, int g, double s, double4* r) {
  const size_t k = g;
  const double* t = a.quad + 6 * k;
  r[0] = make_double4(a.xyz[3 * k], a.xyz[3 * k + 1], a.xyz[3 * k + 2], a.q[k]);
  r[1] = make_double4(a.dip[3 * k], a.dip[3 * k + 1], a.dip[3 * k + 2], s);
  r[2] = make_double4(t[0], t[1], t[2], t[3]);
  r[3] = make_double4(t[4], t[5], a.thole ? a.thole[k] : a.thole_a, __hiloint2double(0, a.mol[k]));
}

// Inverse of a symmetric 3x3 (xx,xy,xz,yy,yz,zz); false unless positive
// definite (leading minors > 0).
__device__ __forceinline__ bool sym_inverse(const double m[6], double inv[6]) {
#pragma clang fp contract(off)   // the same bits in every kernel
  const double a = m[0], b = m[1], c = m[2], d = m[3], e = m[4], f = m[5];
  const double m2 = a * d - b * b;
  const double A = d * f - e * e, B = c * e - b * f, C = b * e - c * d;
  const double det = a * A + b * B + c * C;
  if (!(a > 0.0) || !(m2 > 0.0) || !(det > 0.0)) return false;
  const double id = 1.0 / det;
  inv[0] = A * id;
  inv[1] = B * id;
  inv[2] = C * id;
  inv[3] = (a * f - c * c) * id;
  inv[4] = (b * c - a * e) * id;
  inv[5] = m2 * id;
  return true;
}

// ---------------------------------------------------------------- pair math
// The pair arithmetic with every rounding written out: fused multiply-adds
// are explicit and contraction is off, so the FP32 results of a pair are the
// same in every kernel that evaluates it (a contracted a*b + c*d may fuse
// either product, and which one changes with the code around it).  The
// formulas are those of pairmath.h.
__device__ __forceinline__ double ma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float ma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <typename R>
__device__ __forceinline__ R dot3(const R a[3], const R b[3]) {
#pragma clang fp contract(off)
  return ma(a[2], b[2], ma(a[0], b[0], a[1] * b[1]));
}

template <typename R>
__device__ __forceinline__ void rows3(const R t[6], const R v[3], R o[3]) {
#pragma clang fp contract(off)
  o[0] = ma(t[2], v[2], ma(t[0], v[0], t[1] * v[1]));
  o[1] = ma(t[4], v[2], ma(t[1], v[0], t[3] * v[1]));
  o[2] = ma(t[5], v[2], ma(t[2], v[0], t[4] * v[1]));
}

// Separation and the bare coefficients c0_0..c0_N.
template <typename R, int N>
__device__ __forceinline__ void bare_pair(const double xi[3], const double xj[3], R Rv[3], R& r2,
                                          R& r, R c0[N + 1]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int a = 0; a < 3; ++a) Rv[a] = (R)(xi[a] - xj[a]);
  r2 = dot3<R>(Rv, Rv);
  const R rinv = dev_rsqrt<R>(r2), rinv2 = rinv * rinv;
  r = r2 * rinv;
  c0[0] = rinv;
  if (N >= 1) c0[N >= 1 ? 1 : 0] = rinv * rinv2;
#pragma unroll
  for (int n = 2; n <= N; ++n) c0[n] = R(2 * n - 1) * c0[n - 1] * rinv2;
}

// Thole: x = a r^3 s, tp[n] = 1 - lambda_{2n+1} = P_n(x) e^-x for n = 1..4,
// and with one_minus 1 - tp[n] instead, rounded once.
template <typename R>
__device__ __forceinline__ void thole_pair4(R x, R one_x, bool one_minus, R tp[5]) {
#pragma clang fp contract(off)
  const R e = dev_exp<R>(-x), x2 = x * x;
  const R p3 = ma(x2, R(0.6), one_x);
  const R p4 = ma(x, x2 * R(9.0 / 35.0), ma(x2, R(18.0 / 35.0), one_x));
  tp[0] = R(0);
  if (one_minus) {
    tp[1] = R(1) - e;
    tp[2] = ma(-one_x, e, R(1));
    tp[3] = ma(-p3, e, R(1));
    tp[4] = ma(-p4, e, R(1));
  } else {
    tp[1] = e;
    tp[2] = one_x * e;
    tp[3] = p3 * e;
    tp[4] = p4 * e;
  }
}

// What energy and force of a pair of multipoles share.
template <typename R>
struct PairDots {
  R dri, drj, qir[3], qjr[3], qrri, qrrj, qq, tt;
  __device__ __forceinline__ PairDots(const MP<R>& A, const MP<R>& B, const R Rv[3]) {
#pragma clang fp contract(off)
    dri = dot3<R>(A.d, Rv);
    drj = dot3<R>(B.d, Rv);
    rows3<R>(A.t, Rv, qir);
    rows3<R>(B.t, Rv, qjr);
    qrri = dot3<R>(qir, Rv);
    qrrj = dot3<R>(qjr, Rv);
    qq = dot3<R>(qir, qjr);
    const R off = ma(A.t[4], B.t[4], ma(A.t[1], B.t[1], A.t[2] * B.t[2]));
    tt = ma(R(2), off, ma(A.t[5], B.t[5], ma(A.t[0], B.t[0], A.t[3] * B.t[3])));
  }
};

template <typename R>
__device__ __forceinline__ R pair_energy(const R c[5], const MP<R>& A, const MP<R>& B,
                                         const R Rv[3]) {
#pragma clang fp contract(off)
  const R third = R(1.0 / 3.0);
  const PairDots<R> D(A, B, Rv);
  const R P0 = A.q * B.q;
  const R P1 = dot3<R>(A.d, B.d) + ma(A.q, D.drj, -(B.q * D.dri));
  R P2 = ma(third, ma(B.q, D.qrri, A.q * D.qrrj), -(D.dri * D.drj));
  P2 = ma(R(2.0 / 3.0), dot3<R>(A.d, D.qjr) - dot3<R>(B.d, D.qir), P2);
  P2 = ma(R(2.0 / 9.0), D.tt, P2);
  const R P3 = ma(third, ma(D.drj, D.qrri, -(D.dri * D.qrrj)), R(-4.0 / 9.0) * D.qq);
  const R P4 = R(1.0 / 9.0) * D.qrri * D.qrrj;
  return ma(c[4], P4, ma(c[3], P3, ma(c[2], P2, ma(c[0], P0, c[1] * P1))));
}

template <typename R>
__device__ __forceinline__ void pair_field(const R c[5], const MP<R>& B, const R Rv[3], R E[3]) {
#pragma clang fp contract(off)
  R qjr[3];
  rows3<R>(B.t, Rv, qjr);
  const R drj = dot3<R>(B.d, Rv), qrrj = dot3<R>(qjr, Rv);
  const R rad = ma(c[3], R(1.0 / 3.0) * qrrj, ma(B.q, c[1], drj * c[2]));
#pragma unroll
  for (int a = 0; a < 3; ++a)
    E[a] = ma(Rv[a], rad, -ma(B.d[a], c[1], c[2] * (R(2.0 / 3.0) * qjr[a])));
}

// Force on A of the pair with coefficients c[1..5].  CORR: the damping
// correction of a pair, whose two sums are rounded before they are added.
template <typename R, bool CORR>
__device__ __forceinline__ void pair_force(const R c[6], const MP<R>& A, const MP<R>& B,
                                           const R Rv[3], R F[3]) {
#pragma clang fp contract(off)
  const R third = R(1.0 / 3.0), two3 = R(2.0 / 3.0);
  const PairDots<R> D(A, B, Rv);
  const R P0 = A.q * B.q;
  const R P1 = dot3<R>(A.d, B.d) + ma(A.q, D.drj, -(B.q * D.dri));
  R P2 = ma(-D.dri, D.drj, third * ma(B.q, D.qrri, A.q * D.qrrj));
  P2 = ma(two3, dot3<R>(A.d, D.qjr) - dot3<R>(B.d, D.qir), P2);
  P2 = CORR ? R(2.0 / 9.0) * D.tt + P2 : ma(R(2.0 / 9.0), D.tt, P2);
  const R P3 = ma(third, ma(D.drj, D.qrri, -(D.qrrj * D.dri)), -(R(4.0 / 9.0) * D.qq));
  const R P4 = R(1.0 / 9.0) * D.qrri * D.qrrj;
  R rad = ma(c[4], P3, ma(c[3], P2, ma(c[1], P0, c[2] * P1)));
  if (!CORR) rad = ma(c[5], P4, rad);   // the correction has c5 = 0
  R tjdi[3], tidj[3], tiqjr[3], tjqir[3];
  rows3<R>(B.t, A.d, tjdi);
  rows3<R>(A.t, B.d, tidj);
  rows3<R>(A.t, D.qjr, tiqjr);
  rows3<R>(B.t, D.qir, tjqir);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const R g1 = ma(A.q, B.d[a], -(A.d[a] * B.q));
    R g2 = ma(-A.d[a], D.drj, two3 * ma(D.qir[a], B.q, A.q * D.qjr[a]));
    g2 = ma(two3, tjdi[a] - tidj[a], ma(-D.dri, B.d[a], g2));
    const R u = ma(D.qrri, B.d[a], -(D.qrrj * A.d[a]));
    const R v = ma(D.qir[a], D.drj, -(D.qjr[a] * D.dri));
    const R w = tiqjr[a] + tjqir[a];
    const R g3 = CORR ? ma(two3, v, third * u) - R(4.0 / 9.0) * w
                      : ma(R(-4.0 / 9.0), w, ma(third, u, two3 * v));
    const R g4 = R(2.0 / 9.0) * ma(D.qjr[a], D.qrri, D.qir[a] * D.qrrj);
    F[a] = ma(Rv[a], rad, -ma(c[4], g4, ma(c[3], g3, ma(c[1], g1, c[2] * g2))));
  }
}

// ---------------------------------------------------------------- records
// Records and order-preserving polarizable compaction of one cluster, kClBlock
// sites at a time; returns the number of polarizable sites.  bad: set when a
// polarizability is not positive definite (that site's s stays 0).
__device__ __forceinline__ int cluster_records(const ClusterArgs& a, int base, int n, double4* rec,
                                               int* polsite, int* prank, int* wcount, int* bad) {
  constexpr int W = kClBlock / 64;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int total = 0;
  for (int c0 = 0; c0 < n; c0 += kClBlock) {
    const int i = c0 + t;
    bool is_pol = false;
    double al[6];
    if (i < n) {
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        al[k] = a.alpha[6 * (size_t)(base + i) + k];
        is_pol = is_pol || al[k] != 0.0;
      }
    }
    const unsigned long long m = __ballot(is_pol);
    __syncthreads();
    if (lane == 0) wcount[w] = __popcll(m);
    __syncthreads();
    int before = total;
    for (int k = 0; k < w; ++k) before += wcount[k];
    if (i < n) {
      double s = 0.0;
      int rank = -1;
      if (is_pol) {
        rank = before + lanes_below(m, 0);
        double inv[6];
        if (!sym_inverse(al, inv)) *bad = 1;
        else s = 1.0 / sqrt((al[0] + al[3] + al[5]) / 3.0);
        polsite[rank] = i;
      }
      prank[i] = rank;
      store_rec(a, base + i, s, rec + 4 * i);
    }
    for (int k = 0; k < W; ++k) total += wcount[k];
  }
  return total;
}

// a r^3 of a polarizable pair
template <typename R>
__device__ __forceinline__ R thole_y(const Site<R>& A, const Site<R>& B, R r2, R r) {
#pragma clang fp contract(off)
  return R(fmin(A.th, B.th)) * r2 * r;
}

// ---------------------------------------------------------------- field
// Site j's part of the permanent field at site i (none unless that is
// polarizable) and half the MM energy of the pair.
template <typename R>
__device__ __forceinline__ void field_pair(const Site<R>& A, const Site<R>& B, double E[3],
                                           double& U) {
#pragma clang fp contract(off)
  if (B.mol == A.mol) return;
  R Rv[3], r2, r, c0[5];
  bare_pair<R, 4>(A.x, B.x, Rv, r2, r, c0);
  U += 0.5 * (double)pair_energy<R>(c0, A.M, B.M, Rv);
  if (A.s > 0.0) {
    R cc[5] = {c0[0], c0[1], c0[2], c0[3], R(0)};
    if (B.s > 0.0) {
      const R y = thole_y<R>(A, B, r2, r), sij = R(A.s * B.s);
      R tp[5];
      thole_pair4<R>(y * sij, ma(y, sij, R(1)), false, tp);
#pragma unroll
      for (int k = 1; k <= 3; ++k) cc[k] = ma(-tp[k], c0[k], c0[k]);
    }
    R F[3];
    pair_field<R>(cc, B.M, Rv, F);
    E[0] += (double)F[0];
    E[1] += (double)F[1];
    E[2] += (double)F[2];
  }
}
// Both summed over a site's sixteen lanes.
__device__ __forceinline__ void field_sum(double E[3], double& U) {
#pragma unroll
  for (int k = 0; k < 3; ++k) E[k] = group_sum<kClG>(E[k]);
  U = group_sum<kClG>(U);
}

// ---------------------------------------------------------------- operator
// Damped dipole-dipole coefficients of a pair (every pair of a cluster's
// polarizable sites couples, same molecule included).
template <typename RR>
__device__ __forceinline__ void pair_coef(const RR Rv[3], double ai, double aj, double si,
                                          double sj, RR& c1, RR& c2) {
#pragma clang fp contract(off)
  const RR r2 = dot3<RR>(Rv, Rv);
  const RR rinv = dev_rsqrt<RR>(r2), r = r2 * rinv, rinv2 = rinv * rinv;
  const RR c01 = rinv * rinv2, c02 = RR(3) * c01 * rinv2;
  const RR y = RR(fmin(ai, aj)) * r2 * r, s = RR(si * sj);
  const RR e = dev_exp<RR>(-(y * s));
  c1 = (RR(1) - e) * c01;
  c2 = ma(-ma(y, s, RR(1)), e, RR(1)) * c02;
}

// Field at R of the dipole p
template <typename RR>
__device__ __forceinline__ void dipole_field(RR c1, RR c2, const RR p[3], const RR Rv[3],
                                             RR E[3]) {
#pragma clang fp contract(off)
  const RR a = c2 * dot3<RR>(Rv, p);
#pragma unroll
  for (int k = 0; k < 3; ++k) E[k] = ma(a, Rv[k], -(c1 * p[k]));
}

// The table entry of a pair, whatever its precision.
__device__ __forceinline__ void unpack(double2 c, double& c1, double& c2) { c1 = c.x; c2 = c.y; }
__device__ __forceinline__ void unpack(float2 c, float& c1, float& c2) { c1 = c.x; c2 = c.y; }

// Fields at the rows k0 + m nslot (m < RB; the last row again past it) of
// the dipoles lv, RB rows per pass so that a neighbour's record is read from
// LDS once for all of them; the sixteen lanes' sums, in every lane.  With a
// table (whose diagonal is zero) the loop has no branch, and four steps'
// entries are in flight at once: the trip to L2 bounds it otherwise.
template <typename RR, typename C2, bool TAB, int RB>
__device__ __forceinline__ void dip_rows(const double4* lpos, const double* la, const double4* lv,
                                         const C2* table, int np, int k0, int nslot, int lane,
                                         double f[RB][3]) {
  int kr[RB];
  double px[RB], py[RB], pz[RB];
#pragma unroll
  for (int m = 0; m < RB; ++m) {
    kr[m] = min(k0 + m * nslot, np - 1);
    const double4 p = lpos[kr[m]];
    px[m] = p.x; py[m] = p.y; pz[m] = p.z;
    f[m][0] = f[m][1] = f[m][2] = 0.0;
  }
  auto step = [&](int j, const C2* c) {
    const double4 pj = lpos[j], vj = lv[j];
    const RR v[3] = {(RR)vj.x, (RR)vj.y, (RR)vj.z};
#pragma unroll
    for (int m = 0; m < RB; ++m) {
      if (!TAB && kr[m] == j) continue;
      const RR Rv[3] = {(RR)(px[m] - pj.x), (RR)(py[m] - pj.y), (RR)(pz[m] - pj.z)};
      RR c1, c2;
      if (TAB) {
        unpack(c[m], c1, c2);
      } else {
        const double4 pk = lpos[kr[m]];
        pair_coef<RR>(Rv, la[kr[m]], la[j], pk.w, pj.w, c1, c2);
      }
      RR E[3];
      dipole_field<RR>(c1, c2, v, Rv, E);
      f[m][0] += (double)E[0];
      f[m][1] += (double)E[1];
      f[m][2] += (double)E[2];
    }
  };
  int j = lane;
  if (TAB) {
    constexpr int U = 4;
    for (; j + (U - 1) * kClG < np; j += U * kClG) {
      C2 c[U][RB];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int m = 0; m < RB; ++m) c[u][m] = table[(size_t)kr[m] * np + j + u * kClG];
#pragma unroll
      for (int u = 0; u < U; ++u) step(j + u * kClG, c[u]);
    }
  }
#pragma unroll 1
  for (; j < np; j += kClG) {
    C2 c[RB];
    if (TAB) {
#pragma unroll
      for (int m = 0; m < RB; ++m) c[m] = table[(size_t)kr[m] * np + j];
    }
    step(j, c);
  }
#pragma unroll
  for (int m = 0; m < RB; ++m)
#pragma unroll
    for (int a = 0; a < 3; ++a) f[m][a] = group_sum<kClG>(f[m][a]);
}

// Field of the dipoles lv at this thread's own site (slot + lane nslot).
template <typename RR, typename C2, bool TAB>
__device__ __forceinline__ void dip_field_own(const double4* lpos, const double* la,
                                              const double4* lv, const C2* table, int np, int slot,
                                              int nslot, int lane, double own[3]) {
  own[0] = own[1] = own[2] = 0.0;
#pragma unroll 1
  for (int m = 0; slot + m * nslot < np; m += 2) {
    double f[2][3];
    dip_rows<RR, C2, TAB, 2>(lpos, la, lv, table, np, slot + m * nslot, nslot, lane, f);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (lane == m + u) {
        own[0] = f[u][0]; own[1] = f[u][1]; own[2] = f[u][2];
      }
  }
}

// ---------------------------------------------------------------- solve
// PCG of one cluster by the NT threads of the block.  Sixteen lanes share a
// row of T; rows slot, slot + nslot, ... belong to slot, and its lane m owns
// row slot + m nslot: x, r, z, p and alpha of that site stay in its
// registers, and lv (LDS) holds the vector the operator is applied to.
// al: alpha of this thread's site; E: its field; x: in the first guess, out
// the dipoles.  T64, TR: the FP64 coefficients and those in precision R come
// from their tables.
template <typename R, int NT, typename C2, bool T64, bool TR>
__device__ __forceinline__ void solve_cluster(const double4* lpos, const double* la, double4* lv,
                                              const double2* table, const C2* table_r, int np,
                                              const double al[6], const double4* E, double x[3],
                                              double tol, int max_iter, const BlockSum<NT>& bsum,
                                              int& it, double& rho, int& status) {
#pragma clang fp contract(off)   // the same bits in every kernel
  constexpr int nslot = NT / kClG;
  const int t = threadIdx.x, slot = t / kClG, lane = t % kClG;
  const int k = slot + lane * nslot;
  const bool own = k < np;
  double ai[6] = {0, 0, 0, 0, 0, 0};
  if (own) (void)sym_inverse(al, ai);
  const double zz_stop = (tol / kDebye) * (tol / kDebye) * np;
  it = 0;
  status = 0;
  rho = 0.0;
  int restarts = 0;
  double rz_run = 0.0;            // r.z of the running sequence
  double zz_replace = -1.0;       // see the context solver: one early
  bool fresh = true;              // residual replacement in mixed mode
  double r[3] = {0, 0, 0}, z[3] = {0, 0, 0}, p[3] = {0, 0, 0};
  for (;;) {
    // true residual r = E - T x in FP64, z = alpha r
    __syncthreads();
    if (own) lv[k] = make_double4(x[0], x[1], x[2], 0.0);
    __syncthreads();
    double zz = 0.0, rz = 0.0;
    double f[3];
    dip_field_own<double, double2, T64>(lpos, la, lv, table, np, slot, nslot, lane, f);
    if (own) {
      const double4 e = *E;   // read again: held only here
      double tx[3];
      rows3<double>(ai, x, tx);
      r[0] = e.x - (tx[0] - f[0]);
      r[1] = e.y - (tx[1] - f[1]);
      r[2] = e.z - (tx[2] - f[2]);
      rows3<double>(al, r, z);
      zz = dot3<double>(z, z);
      rz = dot3<double>(r, z);
    }
    bsum(zz, rz);
    rho = kDebye * sqrt(zz / np);
    if (rho <= tol) break;
    if (it >= max_iter || restarts > 8) {
      status = (int)SIBFA_E_NOT_CONVERGED;
      break;
    }
    // a new sequence (p = z) at the start; afterwards the true residual
    // replaces the recurrence one and the sequence goes on (p = z + beta p)
    double beta = fresh ? 0.0 : rz / rz_run;
    if (fresh) {
      if (sizeof(R) == 4) zz_replace = 1e-8 * zz;
    } else {
      ++restarts;
    }
    fresh = false;
    rz_run = rz;
    while (it < max_iter) {
#pragma unroll
      for (int a = 0; a < 3; ++a) p[a] = ma(beta, p[a], z[a]);
      if (own) lv[k] = make_double4(p[0], p[1], p[2], 0.0);
      __syncthreads();
      double pq = 0.0;
      double q[3] = {0, 0, 0};
      dip_field_own<R, C2, TR>(lpos, la, lv, table_r, np, slot, nslot, lane, f);
      if (own) {
        const double4 pv = lv[k];   // p, from LDS: not held through the product
        p[0] = pv.x; p[1] = pv.y; p[2] = pv.z;
        double tp[3];
        rows3<double>(ai, p, tp);
#pragma unroll
        for (int a = 0; a < 3; ++a) q[a] = tp[a] - f[a];
        pq = dot3<double>(p, q);
      }
      bsum(pq);
      if (!(pq > 0.0)) {
        status = (int)SIBFA_E_NOT_SPD;
        break;
      }
      const double gamma = rz_run / pq;
      double zz2 = 0.0, rz2 = 0.0;
      if (own) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          x[a] = ma(gamma, p[a], x[a]);
          r[a] = ma(-gamma, q[a], r[a]);
        }
        rows3<double>(al, r, z);
        zz2 = dot3<double>(z, z);
        rz2 = dot3<double>(r, z);
      }
      bsum(zz2, rz2);
      ++it;
      if (zz2 <= zz_stop) break;
      if (zz2 <= zz_replace) {
        zz_replace = -1.0;
        break;
      }
      beta = rz2 / rz_run;
      rz_run = rz2;
    }
    if (status == (int)SIBFA_E_NOT_SPD) break;
  }
}

// ---------------------------------------------------------------- forces
// Force on the dipole a of two dipoles with coefficients c2, c3.
template <typename R>
__device__ __forceinline__ void same_molecule_force(R c2, R c3, const R a[3], const R b[3],
                                                    const R Rv[3], R F[3]) {
#pragma clang fp contract(off)
  const R da = dot3<R>(a, Rv), db = dot3<R>(b, Rv);
  const R rad = ma(c3, -(da * db), c2 * dot3<R>(a, b));
#pragma unroll
  for (int k = 0; k < 3; ++k)
    F[k] = ma(Rv[k], rad, -(c2 * ma(-da, b[k], -(a[k] * db))));
}

// Force (e^2/A^2) on site A with dipole mui of another site B with dipole
// muj; P is A's multipoles with mui added.
template <typename R>
__device__ __forceinline__ void site_force(const Site<R>& A, const MP<R>& P, const R mui[3],
                                           const Site<R>& B, const R muj[3], double F[3]) {
#pragma clang fp contract(off)
  R Rv[3], r2, r, c0[6];
  bare_pair<R, 5>(A.x, B.x, Rv, r2, r, c0);
  const bool both = A.s > 0.0 && B.s > 0.0;
  const R x = both ? thole_y<R>(A, B, r2, r) * R(A.s * B.s) : R(0);
  R f[3];
  if (B.mol == A.mol) {
    // same molecule: damped mu-mu only
    if (!both) return;
    R l[5];
    thole_pair4<R>(x, R(1) + x, true, l);
    same_molecule_force<R>(l[2] * c0[2], l[3] * c0[3], mui, muj, Rv, f);
    F[0] += (double)f[0];
    F[1] += (double)f[1];
    F[2] += (double)f[2];
    return;
  }
  R cc[6], D[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
#pragma unroll
  for (int k = 0; k < 6; ++k) cc[k] = c0[k];
  const bool damp = both && x < R(50);
  if (damp) {
    R tp[5];
    thole_pair4<R>(x, R(1) + x, false, tp);
#pragma unroll
    for (int k = 1; k <= 4; ++k) {
      D[k] = tp[k] * c0[k];
      cc[k] = ma(-tp[k], c0[k], c0[k]);
    }
  }
  MP<R> Pj = B.M;
#pragma unroll
  for (int k = 0; k < 3; ++k) Pj.d[k] += muj[k];
  pair_force<R, false>(cc, P, Pj, Rv, f);
  F[0] += (double)f[0];
  F[1] += (double)f[1];
  F[2] += (double)f[2];
  if (damp) {
    pair_force<R, true>(D, A.M, B.M, Rv, f);
    F[0] += (double)f[0];
    F[1] += (double)f[1];
    F[2] += (double)f[2];
  }
}

__device__ __forceinline__ double quiet_nan() { return __longlong_as_double(0x7ff8000000000000ll); }

// mu and forces zero, E_pol undefined (bad polarizabilities, too many
// polarizable sites), or no polarizable site (status 0, E_pol 0).
template <int NT>
__device__ __forceinline__ void no_solution(const ClusterArgs& a, int c, int base, int n, int st) {
  for (int i = threadIdx.x; i < 3 * n; i += NT) a.mu[3 * (size_t)base + i] = 0.0;
  if (threadIdx.x == 0) {
    a.e_pol[c] = st != 0 ? quiet_nan() : 0.0;
    a.iters[c] = 0;
    a.rms[c] = 0.0;
    a.status[c] = st;
  }
}

// ---------------------------------------------------------------- small clusters
template <typename R>
struct SmallLds {
  using C2 = typename std::conditional<sizeof(R) == 8, double2, float2>::type;
  double4 rec[4 * kClSmall];
  double4 lmu[kClSmall], lpos[kClSmall], lv[kClSmall], lE[kClSmall];
  C2 table[kClSmallTable * kClSmallTable];
  double la[kClSmall];
  double sh[2 * (kClBlock / 64)];
  int polsite[kClSmall], prank[kClSmall], wcount[kClBlock / 64], bad;
};

// Clusters first, first + stride, ... : one workgroup of kClBlock threads
// takes a small cluster through records, field, solve and forces without
// leaving its LDS, and passes over the large ones.
template <typename R>
__device__ __forceinline__ void small_clusters(const ClusterArgs& a, SmallLds<R>& l, int first,
                                               int stride) {
  using C2 = typename SmallLds<R>::C2;
  double4 *rec = l.rec, *lmu = l.lmu, *lpos = l.lpos, *lv = l.lv, *lE = l.lE;
  double* la = l.la;
  int *polsite = l.polsite, *prank = l.prank;
  C2* table = l.table;
  const BlockSum<kClBlock> bsum{l.sh};
  constexpr int nslot = kClTile;
  const int t = threadIdx.x, slot = t / kClG, lane = t % kClG;
  for (int c = first; c < a.nclusters; c += stride) {
    int base, n;
    if (!cluster_range(a, c, base, n)) {
      if (t == 0) {
        a.status[c] = (int)SIBFA_E_ARG;
        a.e_elec[c] = a.e_pol[c] = quiet_nan();
        a.iters[c] = 0;
        a.rms[c] = 0.0;
      }
      continue;
    }
    if (n > kClSmall) continue;
    __syncthreads();
    if (t == 0) l.bad = 0;
    const int np = cluster_records(a, base, n, rec, polsite, prank, l.wcount, &l.bad);
    __syncthreads();
    double U = 0.0;
    for (int i = slot; i < n; i += nslot) {
      Site<R> A;
      load_rec<R>(rec, i, A);
      double E[3] = {0.0, 0.0, 0.0}, u = 0.0;
      for (int j = lane; j < n; j += kClG) {
        Site<R> B;
        load_rec<R>(rec, j, B);
        field_pair<R>(A, B, E, u);
      }
      field_sum(E, u);
      if (lane == 0) {
        U += u;
        lE[i] = make_double4(E[0], E[1], E[2], 0.0);
        lmu[i] = make_double4(0.0, 0.0, 0.0, 0.0);
      }
    }
    if (t < np) {
      const double4 p = rec[4 * polsite[t]];
      lpos[t] = make_double4(p.x, p.y, p.z, rec[4 * polsite[t] + 1].w);
      la[t] = rec[4 * polsite[t] + 3].z;
    }
    bsum(U);
    if (t == 0) a.e_elec[c] = kCoulomb * U;
    const int st0 = l.bad ? (int)SIBFA_E_ARG : 0;
    if (st0 != 0 || np == 0) {
      no_solution<kClBlock>(a, c, base, n, st0);
    } else {
      const bool tab = np <= kClSmallTable;
      if (tab) {
        for (int e = t; e < np * np; e += kClBlock) {
          const int k = e / np, j = e - k * np;
          R c1 = R(0), c2 = R(0);
          if (j != k) {
            const double4 pk = lpos[k], pj = lpos[j];
            const R Rv[3] = {(R)(pk.x - pj.x), (R)(pk.y - pj.y), (R)(pk.z - pj.z)};
            pair_coef<R>(Rv, la[k], la[j], pk.w, pj.w, c1, c2);
          }
          C2 v;
          v.x = c1; v.y = c2;
          table[e] = v;
        }
      }
      const int k = slot + lane * nslot;
      const bool own = k < np;
      const int ks = own ? polsite[k] : 0;
      double al[6] = {0, 0, 0, 0, 0, 0}, x[3] = {0, 0, 0};
      const double4* E = lE + ks;
      if (own) {
#pragma unroll
        for (int m = 0; m < 6; ++m) al[m] = a.alpha[6 * (size_t)(base + ks) + m];
        if (a.warm && a.warm[c]) {
#pragma unroll
          for (int m = 0; m < 3; ++m) x[m] = a.mu[3 * (size_t)(base + ks) + m];
        } else {
          const double e[3] = {E->x, E->y, E->z};
          rows3<double>(al, e, x);
        }
      }
      constexpr bool same = sizeof(R) == 8;   // one table serves both precisions
      const double2* t64 = same ? reinterpret_cast<const double2*>(table) : nullptr;
      int it, status;
      double rho;
      if (tab)
        solve_cluster<R, kClBlock, C2, same, true>(lpos, la, lv, t64, table, np, al, E, x, a.tol,
                                                   a.max_iter, bsum, it, rho, status);
      else
        solve_cluster<R, kClBlock, C2, false, false>(lpos, la, lv, nullptr, nullptr, np, al, E, x,
                                                     a.tol, a.max_iter, bsum, it, rho, status);
      double me = 0.0;
      if (own) {
        lmu[ks] = make_double4(x[0], x[1], x[2], 0.0);
        const double e[3] = {E->x, E->y, E->z};
        me = dot3<double>(x, e);
      }
      bsum(me);
      if (t == 0) {
        a.e_pol[c] = -0.5 * kCoulomb * me;
        a.iters[c] = it;
        a.rms[c] = rho;
        a.status[c] = status;
      }
      __syncthreads();
      for (int i = t; i < n; i += kClBlock) {
        const double4 m = lmu[i];
        double* o = a.mu + 3 * (size_t)(base + i);
        o[0] = m.x; o[1] = m.y; o[2] = m.z;
      }
    }
    if (!a.forces) continue;
    if (st0 != 0) {
      for (int i = t; i < 3 * n; i += kClBlock) a.forces[3 * (size_t)base + i] = 0.0;
      continue;
    }
    auto mu = [&](int j, R m[3]) {
      const double4 v = lmu[j];
      m[0] = (R)v.x; m[1] = (R)v.y; m[2] = (R)v.z;
    };
    for (int i = slot; i < n; i += nslot) {
      Site<R> A;
      load_rec<R>(rec, i, A);
      R mui[3], muj[3];
      mu(i, mui);
      MP<R> P = A.M;
      for (int k = 0; k < 3; ++k) P.d[k] += mui[k];
      double F[3] = {0.0, 0.0, 0.0};
      for (int j = lane; j < n; j += kClG) {
        if (j == i) continue;
        Site<R> B;
        load_rec<R>(rec, j, B);
        mu(j, muj);
        site_force<R>(A, P, mui, B, muj, F);
      }
      for (int k = 0; k < 3; ++k) F[k] = group_sum<kClG>(F[k]);
      if (lane == 0)
        for (int k = 0; k < 3; ++k) a.forces[3 * (size_t)(base + i) + k] = kCoulomb * F[k];
    }
  }
}

// The small clusters of a batch in a launch of their own.  700 clusters of 2
// to 8 waters (FP64): 104 us for the whole call, against 192 us with one launch
// per stage, dipole coefficients re-evaluated in every product and records
// gathered from memory; one dimer 39 us against 58.
template <typename R>
__global__ __launch_bounds__(kClBlock) void k_cl_small(ClusterArgs a) {
  __shared__ SmallLds<R> l;
  if (a.apart && !*a.apart) return;
  small_clusters<R>(a, l, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------- large clusters
// The large clusters of the batch in order, -1 after the last, and whether the
// small ones run apart, by one workgroup.
__device__ __forceinline__ void list_large(const ClusterArgs& a, int* wcount) {
  constexpr int W = kClBlock / 64;
  __shared__ BatchCost sum;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t == 0) sum = BatchCost{};
  int total = 0;
  for (int c0 = 0; c0 < a.nclusters; c0 += kClBlock) {
    const int c = c0 + t;
    int base, n;
    const bool on = c < a.nclusters && cluster_range(a, c, base, n), big = on && n > kClSmall;
    const unsigned long long m = __ballot(big);
    __syncthreads();
    if (lane == 0) wcount[w] = __popcll(m);
    if (on) {
      atomicAdd(big ? &sum.nl : &sum.ns, 1);
      atomicAdd(big ? &sum.cl : &sum.cs, cluster_cost(n));
      if (big) atomicMax(&sum.ml, cluster_cost(n));
    }
    __syncthreads();
    int before = total;
    for (int k = 0; k < w; ++k) before += wcount[k];
    if (big) a.list[lanes_below(m, before)] = c;
    for (int k = 0; k < W; ++k) total += wcount[k];
  }
  for (int k = total + t; k < a.nclusters; k += kClBlock) a.list[k] = -1;
  if (t == 0) *a.apart = small_apart(sum) ? 1 : 0;
}

// Clusters of a batch whose sizes the host does not know (a.list) are all
// looked at, and the last workgroup writes the list for the other kernels.
__global__ __launch_bounds__(kClBlock) void k_cl_prep(ClusterArgs a, int count) {
  __shared__ int wcount[kClBlock / 64], bad;
  int nwg = gridDim.x;
  if (a.list && (int)blockIdx.x == --nwg) {
    list_large(a, wcount);
    return;
  }
  for (int b = blockIdx.x; b < count; b += nwg) {
    const int c = a.list ? b : a.large[b];
    int base, n;
    if (!large_cluster(a, c, base, n)) continue;
    __syncthreads();
    if (threadIdx.x == 0) bad = 0;
    const int np = cluster_records(a, base, n, a.rec + 4 * (size_t)base, a.polsite + base,
                                   a.prank + base, wcount, &bad);
    __syncthreads();
    if (threadIdx.x == 0) {
      a.npol[c] = np;
      a.status[c] = (bad || np > kClMaxPol) ? (int)SIBFA_E_ARG : 0;
    }
  }
}

// A chunk of a cluster's sites in LDS, in the pairs' precision, for the field
// and force sums of sixteen sites.  With every lane reading and converting its
// neighbour's record from memory (four 32-byte loads a pair, sixteen sites'
// records per wavefront) many clusters took longer than the pairs' arithmetic:
// 1,000 clusters of 64 waters, field and forces 1,586 + 1,588 -> 407 + 590 us
// (mixed), 1,622 + 1,575 -> 648 + 1,090 (FP64); 1,000 of 13 to 20 waters (mixed)
// 144 + 133 -> 66 + 71 us; 48 of 64 waters as a whole 417 -> 305 us.
// An odd number of 16-byte words per site: the sixteen lanes' reads fall in
// different banks.
constexpr int kClStage = 128;
template <typename R>
struct alignas(16) StagedSite {
  double x[3], s;
  MP<R> M;
  double th;
  R mu[3];
  int mol, pad[4];
};
static_assert(sizeof(StagedSite<float>) / 16 % 2 == 1 && sizeof(StagedSite<double>) / 16 % 2 == 1,
              "bank spread of the staged sites");

// Sites [j0, j0 + count) of a cluster, with their dipoles where gmu is given.
template <typename R>
__device__ __forceinline__ void stage_sites(const double4* rec, const double* gmu, int j0,
                                            int count, StagedSite<R>* l) {
  const int t = threadIdx.x;
  __syncthreads();   // the chunk before is read
  if (t < count) {
    Site<R> S;
    load_rec<R>(rec, j0 + t, S);
    StagedSite<R>& o = l[t];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      o.x[k] = S.x[k];
      o.mu[k] = gmu ? (R)gmu[3 * (j0 + t) + k] : R(0);
    }
    o.s = S.s;
    o.M = S.M;
    o.th = S.th;
    o.mol = S.mol;
  }
  __syncthreads();
}
template <typename R>
__device__ __forceinline__ void staged_site(const StagedSite<R>& o, Site<R>& S) {
#pragma unroll
  for (int k = 0; k < 3; ++k) S.x[k] = o.x[k];
  S.M = o.M;
  S.s = o.s;
  S.th = o.th;
  S.mol = o.mol;
}

// gridDim.y workgroups per cluster walk its sites, sixteen at a time
// (blockIdx.z = 0: field and MM energy), or its rows of the coefficient
// table (blockIdx.z = 1).
template <typename R>
__global__ __launch_bounds__(kClBlock) void k_cl_field(ClusterArgs a, int count) {
  __shared__ StagedSite<R> l[kClStage];
  const int t = threadIdx.x, slot = t / kClG, lane = t % kClG;
  for (int b = blockIdx.x, c; (c = cluster_at(a, b, count)) >= 0; b += gridDim.x) {
    int base, n;
    if (!large_cluster(a, c, base, n)) continue;
    const double4* rec = a.rec + 4 * (size_t)base;
    if (blockIdx.z == 0) {
      for (int i0 = blockIdx.y * kClTile; i0 < n; i0 += gridDim.y * kClTile) {
        const int i = i0 + slot;
        Site<R> A;
        load_rec<R>(rec, min(i, n - 1), A);
        double E[3] = {0.0, 0.0, 0.0}, u = 0.0;
        for (int j0 = 0; j0 < n; j0 += kClStage) {
          const int m = min(kClStage, n - j0);
          stage_sites<R>(rec, nullptr, j0, m, l);
          if (i >= n) continue;
          for (int j = lane; j < m; j += kClG) {
            Site<R> B;
            staged_site<R>(l[j], B);
            field_pair<R>(A, B, E, u);
          }
        }
        field_sum(E, u);
        if (lane == 0 && i < n) {
          a.usite[base + i] = u;
          const int k = a.prank[base + i];
          if (k >= 0) a.E0[base + k] = make_double4(E[0], E[1], E[2], 0.0);
        }
      }
      continue;
    }
    const long long off = a.coef_off[c];
    const int np = a.npol[c];
    if (off < 0 || np > kClMaxPol) continue;
    const int* ps = a.polsite + base;
    for (int k = blockIdx.y * kClTile + slot; k < np; k += gridDim.y * kClTile) {
      const int sk = ps[k];
      const double4 pk = rec[4 * sk];
      const double s = rec[4 * sk + 1].w, th = rec[4 * sk + 3].z;
      for (int j = lane; j < np; j += kClG) {
        const size_t e = (size_t)off + (size_t)k * np + j;
        if (j == k) {   // no coupling of a site with itself
          a.coef[e] = make_double2(0.0, 0.0);
          if (sizeof(R) == 4) a.coef32[e] = make_float2(0.f, 0.f);
          continue;
        }
        const int sj = ps[j];
        const double4 pj = rec[4 * sj];
        const double sjv = rec[4 * sj + 1].w, thj = rec[4 * sj + 3].z;
        const double Rd[3] = {pk.x - pj.x, pk.y - pj.y, pk.z - pj.z};
        double c1, c2;
        pair_coef<double>(Rd, th, thj, s, sjv, c1, c2);
        a.coef[e] = make_double2(c1, c2);
        if (sizeof(R) == 4) {
          const float Rf[3] = {(float)Rd[0], (float)Rd[1], (float)Rd[2]};
          float f1, f2;
          pair_coef<float>(Rf, th, thj, s, sjv, f1, f2);
          a.coef32[e] = make_float2(f1, f2);
        }
      }
    }
  }
}

template <typename R> __device__ __forceinline__ auto coef_table(const ClusterArgs& a);
template <> __device__ __forceinline__ auto coef_table<double>(const ClusterArgs& a) { return a.coef; }
template <> __device__ __forceinline__ auto coef_table<float>(const ClusterArgs& a) { return a.coef32; }

// Solves of the large clusters by the first gridDim.x - nsmall workgroups
// (TAB: of those with a coefficient table, otherwise of those without); the
// last nsmall run the batch's small clusters beside them with their first
// kClBlock threads, since the solves leave most of the GPU idle.  A solve is
// a chain of matrix products by one workgroup: with 48 clusters of 2 to 64
// waters (mixed precision) the launch takes 185 us, against 680 us when 256
// threads re-evaluated the coefficients in every product (field 350 -> 23,
// forces 510 -> 30 us), and the whole call 1.57 -> 0.25 ms.
template <typename R>
struct SolveLds {
  double4 lpos[kClMaxPol], lv[kClMaxPol];
  double la[kClMaxPol];
  double sh[2 * (kClSolveBlock / 64)];
};

template <typename R, bool TAB>
__global__ __launch_bounds__(kClSolveBlock) void k_cl_solve(ClusterArgs a, int count, int nsmall) {
  using C2 = typename SmallLds<R>::C2;
  constexpr size_t kLds = sizeof(SmallLds<R>) > sizeof(SolveLds<R>) ? sizeof(SmallLds<R>)
                                                                    : sizeof(SolveLds<R>);
  __shared__ __align__(32) char lds[kLds];
  const int nlarge = gridDim.x - nsmall;
  if ((int)blockIdx.x >= nlarge) {
    if (a.apart && *a.apart) return;
    // The other wavefronts end here, by a scalar branch, before the barriers of
    // the first: s_barrier waits for the wavefronts of a workgroup that have not
    // ended, so those synchronise among themselves.  Kept alive to come to every
    // barrier instead, they cost 40 + 40 clusters of 2 to 12 and of 20 waters 164
    // -> 180 us (mixed).
    if (__builtin_amdgcn_readfirstlane(threadIdx.x) >= kClBlock) return;
    small_clusters<R>(a, *reinterpret_cast<SmallLds<R>*>(lds), blockIdx.x - nlarge, nsmall);
    return;
  }
  SolveLds<R>& l = *reinterpret_cast<SolveLds<R>*>(lds);
  double4 *lpos = l.lpos, *lv = l.lv;
  double* la = l.la;
  const BlockSum<kClSolveBlock> bsum{l.sh};
  constexpr int nslot = kClSolveBlock / kClG;
  const int t = threadIdx.x, slot = t / kClG, lane = t % kClG;
  for (int b = blockIdx.x, c; (c = cluster_at(a, b, count)) >= 0; b += nlarge) {
    int base, n;
    if (!large_cluster(a, c, base, n)) continue;
    const long long off = a.coef_off ? a.coef_off[c] : -1;
    if ((off >= 0) != TAB) continue;
    const int np = a.npol[c], st0 = a.status[c];
    __syncthreads();   // every thread has the status before it is rewritten
    double U = 0.0;
    for (int i = t; i < n; i += kClSolveBlock) U += a.usite[base + i];
    bsum(U);
    if (t == 0) a.e_elec[c] = kCoulomb * U;
    if (st0 != 0 || np == 0) {
      no_solution<kClSolveBlock>(a, c, base, n, st0);
      continue;
    }
    const double4* rec = a.rec + 4 * (size_t)base;
    if (t < np) {
      const int i = a.polsite[base + t];
      const double4 p = rec[4 * i];
      lpos[t] = make_double4(p.x, p.y, p.z, rec[4 * i + 1].w);
      la[t] = rec[4 * i + 3].z;
    }
    const int k = slot + lane * nslot;
    const bool own = k < np;
    const size_t g = base + (own ? a.polsite[base + k] : 0);
    double al[6] = {0, 0, 0, 0, 0, 0}, x[3] = {0, 0, 0};
    const double4* E = a.E0 + base + (own ? k : 0);
    if (own) {
#pragma unroll
      for (int m = 0; m < 6; ++m) al[m] = a.alpha[6 * g + m];
      if (a.warm && a.warm[c]) {
#pragma unroll
        for (int m = 0; m < 3; ++m) x[m] = a.mu[3 * g + m];
      } else {
        const double e[3] = {E->x, E->y, E->z};
        rows3<double>(al, e, x);
      }
    }
    const double2* t64 = TAB ? a.coef + off : nullptr;
    const C2* tr = TAB ? coef_table<R>(a) + off : nullptr;
    int it, status;
    double rho;
    solve_cluster<R, kClSolveBlock, C2, TAB, TAB>(lpos, la, lv, t64, tr, np, al, E, x, a.tol,
                                                  a.max_iter, bsum, it, rho, status);
    double me = 0.0;
    if (own) {
      const double e[3] = {E->x, E->y, E->z};
      me = dot3<double>(x, e);
    }
    bsum(me);
    for (int i = t; i < n; i += kClSolveBlock)
      if (a.prank[base + i] < 0)
        for (int m = 0; m < 3; ++m) a.mu[3 * (size_t)(base + i) + m] = 0.0;
    if (own)
      for (int m = 0; m < 3; ++m) a.mu[3 * g + m] = x[m];
    if (t == 0) {
      a.e_pol[c] = -0.5 * kCoulomb * me;
      a.iters[c] = it;
      a.rms[c] = rho;
      a.status[c] = status;
    }
  }
}

template <typename R>
__global__ __launch_bounds__(kClBlock) void k_cl_force(ClusterArgs a, int count) {
  __shared__ StagedSite<R> l[kClStage];
  const int t = threadIdx.x, slot = t / kClG, lane = t % kClG;
  for (int b = blockIdx.x, c; (c = cluster_at(a, b, count)) >= 0; b += gridDim.x) {
    int base, n;
    if (!large_cluster(a, c, base, n)) continue;
    const bool zero = a.status[c] == (int)SIBFA_E_ARG;
    const double* gmu = a.mu + 3 * (size_t)base;
    const double4* rec = a.rec + 4 * (size_t)base;
    for (int i0 = blockIdx.y * kClTile; i0 < n; i0 += gridDim.y * kClTile) {
      const int i = i0 + slot, is = min(i, n - 1);
      double F[3] = {0.0, 0.0, 0.0};
      Site<R> A;
      load_rec<R>(rec, is, A);
      const R mui[3] = {(R)gmu[3 * is], (R)gmu[3 * is + 1], (R)gmu[3 * is + 2]};
      MP<R> P = A.M;
#pragma unroll
      for (int k = 0; k < 3; ++k) P.d[k] += mui[k];
      for (int j0 = 0; j0 < (zero ? 0 : n); j0 += kClStage) {
        const int m = min(kClStage, n - j0);
        stage_sites<R>(rec, gmu, j0, m, l);
        if (i >= n) continue;
        for (int j = lane; j < m; j += kClG) {
          if (j0 + j == i) continue;
          Site<R> B;
          staged_site<R>(l[j], B);
          site_force<R>(A, P, mui, B, l[j].mu, F);
        }
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) F[k] = group_sum<kClG>(F[k]);
      if (lane == 0 && i < n)
        for (int k = 0; k < 3; ++k) a.forces[3 * (size_t)(base + i) + k] = kCoulomb * F[k];
    }
  }
}

}  // namespace sibfa

using namespace sibfa;

// Device memory of sibfa_batch_clusters_noalloc: the batch scratch arrays
// for SIBFA_BATCH_NOALLOC_MAX_SITES sites and SIBFA_BATCH_NOALLOC_MAX_CLUSTERS
// clusters, carved as by carve() below (every region rounded up to 256
// bytes).  Each device the library runs on holds its own copy for the life
// of the process; calls on one device share it.
namespace {
constexpr size_t kNaSites = SIBFA_BATCH_NOALLOC_MAX_SITES;
constexpr size_t kNaClusters = SIBFA_BATCH_NOALLOC_MAX_CLUSTERS;
constexpr size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t kNaBytes =
    a256((kNaClusters + 1) * sizeof(int)) + 3 * a256(kNaClusters * sizeof(int)) +
    a256(kNaClusters * sizeof(long long)) + a256(sizeof(int)) + 2 * a256(kNaSites * sizeof(int)) +
    a256(kNaSites * sizeof(double)) + 5 * a256(kNaSites * sizeof(double4));
}  // namespace

static __device__ __align__(256) unsigned char scratch[kNaBytes];

struct sibfa_batch_s {
  int device = 0;
  hipStream_t stream = nullptr;
  sibfa_alloc_fn af = nullptr;
  sibfa_free_fn ff = nullptr;
  void* user = nullptr;
  std::string err;
  size_t cap_sites = 0, cap_clusters = 0;
  void* scratch = nullptr;   // one device allocation holding every array
  // coefficient tables of the large clusters, at most kClTableBytes in all;
  // table_refused: the smallest size that there was no memory for (0: none)
  void* table = nullptr;
  size_t table_bytes = 0, table_refused = 0;
  // pinned staging of table starts, offsets, warm flags and large clusters
  char* h_stage = nullptr;
  size_t h_cap = 0;          // bytes
  hipEvent_t staged = nullptr;
  bool staged_pending = false;
  ClusterArgs args{};
};

namespace {

sibfa_status bfail(sibfa_batch b, sibfa_status s, const std::string& msg) {
  if (b) b->err = msg;
  return s;
}

void* balloc(sibfa_batch b, size_t bytes) {
  if (b->af) return b->af(bytes, b->user);
  void* p = nullptr;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();   // a failed allocation is handled by the caller
  return nullptr;
}

void bfree(sibfa_batch b, void* p) {
  if (!p) return;
  if (b->ff) b->ff(p, b->user);
  else (void)hipFree(p);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Carves the scratch arrays for `sites` sites and `clusters` clusters out of
// one allocation (or only measures it when base is null).
size_t carve(char* base, size_t sites, size_t clusters, ClusterArgs* a) {
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + o : nullptr;
    o += align256(bytes);
    return p;
  };
  // the first four are uploaded together (see sibfa_batch_clusters)
  char* coef_off = take(clusters * sizeof(long long));
  char* off = take((clusters + 1) * sizeof(int));
  char* warm = take(clusters * sizeof(int));
  char* large = take(clusters * sizeof(int));
  char* npol = take(clusters * sizeof(int));
  char* apart = take(sizeof(int));
  char* polsite = take(sites * sizeof(int));
  char* prank = take(sites * sizeof(int));
  char* usite = take(sites * sizeof(double));
  char* rec = take(4 * sites * sizeof(double4));
  char* E0 = take(sites * sizeof(double4));
  if (a) {
    a->coef_off = reinterpret_cast<long long*>(coef_off);
    a->off = reinterpret_cast<int*>(off);
    a->warm = reinterpret_cast<int*>(warm);
    a->large = reinterpret_cast<int*>(large);
    a->npol = reinterpret_cast<int*>(npol);
    a->apart = reinterpret_cast<int*>(apart);
    a->polsite = reinterpret_cast<int*>(polsite);
    a->prank = reinterpret_cast<int*>(prank);
    a->usite = reinterpret_cast<double*>(usite);
    a->rec = reinterpret_cast<double4*>(rec);
    a->E0 = reinterpret_cast<double4*>(E0);
  }
  return o;
}

#define BHIP(call)                                                                  \
  do {                                                                              \
    hipError_t e_ = (call);                                                         \
    if (e_ != hipSuccess) return bfail(b, SIBFA_E_DEVICE, hipGetErrorString(e_));   \
  } while (0)

// Which kernels a batch needs: gs workgroups for its small clusters, run apart
// or beside the large solves (both: the device decides, a.apart), and gx for the
// `large` entries of the list of large ones, tiles for each of them; bare: some
// have no coefficient table.  Any numbers of workgroups >= 1 give the same
// results.
struct BatchPlan {
  bool apart = false, beside = false, bare = false;
  int gs = 0, large = 0, gx = 0, tiles = 1;
};
template <typename R>
void launch_batch(const ClusterArgs& a, const BatchPlan& p, hipStream_t st) {
  const dim3 b(kClBlock), bs(kClSolveBlock);
  if (p.large > 0)
    hipLaunchKernelGGL(k_cl_prep, dim3(a.list ? p.large + 1 : p.gx), b, 0, st, a, p.large);
  if (p.apart) hipLaunchKernelGGL(k_cl_small<R>, dim3(p.gs), b, 0, st, a);
  if (p.large <= 0) return;
  hipLaunchKernelGGL(k_cl_field<R>, dim3(p.gx, p.tiles, a.coef_off ? 2 : 1), b, 0, st, a, p.large);
  const int gs = p.beside ? p.gs : 0;
  if (a.coef_off)
    hipLaunchKernelGGL((k_cl_solve<R, true>), dim3(p.gx + gs), bs, 0, st, a, p.large, gs);
  if (p.bare) {
    const int g2 = a.coef_off ? 0 : gs;   // the small clusters run once
    hipLaunchKernelGGL((k_cl_solve<R, false>), dim3(p.gx + g2), bs, 0, st, a, p.large, g2);
  }
  if (a.forces) hipLaunchKernelGGL(k_cl_force<R>, dim3(p.gx, p.tiles), b, 0, st, a, p.large);
}

// Bound on the coefficient tables kept with an executor.  They are reserved by
// the clusters' sites (the host does not know how many are polarizable, 192 of
// the 320 of 64 waters): 512 MB for 327 clusters of 64 waters in FP64 and 218
// in mixed precision.  Clusters past the bound re-evaluate their coefficients in
// every product.
constexpr size_t kClTableBytes = (size_t)512 << 20;

// Room for `bytes` of tables, or as much of it as there is memory for: more
// than that, to grow into, the exact size, or the table that there was.
// Growing waits for the stream, where an earlier batch may read the old table,
// so a size that was refused is not asked for again.
sibfa_status grow_table(sibfa_batch b, size_t bytes) {
  if (bytes <= b->table_bytes || (b->table_refused && bytes >= b->table_refused))
    return SIBFA_OK;
  BHIP(hipStreamSynchronize(b->stream));
  const size_t old = b->table_bytes;
  bfree(b, b->table);
  b->table = nullptr;
  b->table_bytes = 0;
  size_t refused = 0;
  for (size_t want : {std::min(kClTableBytes, std::max(bytes, 2 * old)), bytes, old}) {
    if (want == 0 || want == refused) continue;
    if ((b->table = balloc(b, want))) {
      b->table_bytes = want;
      break;
    }
    refused = want;
  }
  if (b->table_bytes < bytes) b->table_refused = bytes;
  return SIBFA_OK;
}

}  // namespace

extern "C" {

sibfa_status sibfa_batch_create(sibfa_batch* out, int device, void* hip_stream,
                                sibfa_alloc_fn alloc_fn, sibfa_free_fn free_fn, void* user) {
  if (!out) return SIBFA_E_ARG;
  *out = nullptr;
  if ((alloc_fn == nullptr) != (free_fn == nullptr)) return SIBFA_E_ARG;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return SIBFA_E_DEVICE;
  if (hipSetDevice(device) != hipSuccess) return SIBFA_E_DEVICE;
  sibfa_batch b = new sibfa_batch_s();
  b->device = device;
  b->stream = static_cast<hipStream_t>(hip_stream);
  b->af = alloc_fn;
  b->ff = free_fn;
  b->user = user;
  if (hipEventCreateWithFlags(&b->staged, hipEventDisableTiming) != hipSuccess) {
    delete b;
    return SIBFA_E_DEVICE;
  }
  *out = b;
  return SIBFA_OK;
}

void sibfa_batch_destroy(sibfa_batch b) {
  if (!b) return;
  (void)hipSetDevice(b->device);
  (void)hipStreamSynchronize(b->stream);
  bfree(b, b->scratch);
  bfree(b, b->table);
  if (b->h_stage) (void)hipHostFree(b->h_stage);
  if (b->staged) (void)hipEventDestroy(b->staged);
  delete b;
}

const char* sibfa_batch_last_error(sibfa_batch b) { return b ? b->err.c_str() : "null batch"; }

sibfa_status sibfa_batch_clusters(sibfa_batch b, int n_clusters, const int* site_offsets,
                                  const int* warm_start, const double* xyz, const int32_t* mol,
                                  const double* q, const double* dip, const double* quad,
                                  const double* alpha, const double* thole,
                                  const sibfa_params* params, double* mu, double* forces,
                                  double* e_pol, double* e_elec, int* iterations,
                                  double* rms_debye, int* status) {
  if (!b) return SIBFA_E_ARG;
  if (n_clusters <= 0 || !site_offsets)
    return bfail(b, SIBFA_E_ARG, "n_clusters > 0 and site_offsets required");
  if (!xyz || !mol || !q || !dip || !quad || !alpha || !params || !mu || !e_pol || !e_elec ||
      !iterations || !rms_debye || !status)
    return bfail(b, SIBFA_E_ARG, "a required array is NULL");
  if (!(params->tol_debye > 0.0) || params->max_iter < 1 || !(params->thole_a > 0.0) ||
      (params->precision != SIBFA_FP64 && params->precision != SIBFA_MIXED))
    return bfail(b, SIBFA_E_ARG, "tol_debye > 0, max_iter >= 1, thole_a > 0 and a valid precision required");
  if (site_offsets[0] != 0) return bfail(b, SIBFA_E_ARG, "site_offsets[0] must be 0");
  for (int c = 0; c < n_clusters; ++c) {
    const int nc = site_offsets[c + 1] - site_offsets[c];
    if (nc < 1 || nc > kClMaxSites)
      return bfail(b, SIBFA_E_ARG, "every cluster needs 1 to SIBFA_BATCH_MAX_SITES sites");
  }
  const size_t n = (size_t)site_offsets[n_clusters];
  BHIP(hipSetDevice(b->device));
  if (b->staged_pending) {   // the previous upload still reads the staging
    BHIP(hipEventSynchronize(b->staged));
    b->staged_pending = false;
  }
  if (n > b->cap_sites || (size_t)n_clusters > b->cap_clusters) {
    // grow: earlier batches on the stream may still read the old arrays
    BHIP(hipStreamSynchronize(b->stream));
    const size_t sites = std::max(n, 2 * b->cap_sites);
    const size_t clusters = std::max<size_t>(n_clusters, std::max<size_t>(64, 2 * b->cap_clusters));
    bfree(b, b->scratch);
    b->scratch = nullptr;
    b->cap_sites = b->cap_clusters = 0;
    void* p = balloc(b, carve(nullptr, sites, clusters, nullptr));
    if (!p) return bfail(b, SIBFA_E_NOMEM, "batch scratch allocation failed");
    b->scratch = p;
    b->cap_sites = sites;
    b->cap_clusters = clusters;
  }
  ClusterArgs a{};
  carve(static_cast<char*>(b->scratch), b->cap_sites, b->cap_clusters, &a);
  // one upload: the staging mirrors the first arrays of the scratch
  const char* dev0 = static_cast<const char*>(b->scratch);
  const size_t o_off = reinterpret_cast<const char*>(a.off) - dev0,
               o_warm = reinterpret_cast<const char*>(a.warm) - dev0,
               o_large = reinterpret_cast<const char*>(a.large) - dev0;
  const size_t need = o_large + (size_t)n_clusters * sizeof(int);
  if (need > b->h_cap) {
    if (b->h_stage) BHIP(hipHostFree(b->h_stage));
    b->h_stage = nullptr;
    b->h_cap = 0;
    BHIP(hipHostMalloc(reinterpret_cast<void**>(&b->h_stage), need, hipHostMallocDefault));
    b->h_cap = need;
  }
  const bool mix = params->precision == SIBFA_MIXED;
  const size_t pair_bytes = sizeof(double2) + (mix ? sizeof(float2) : 0);
  long long* h_coef = reinterpret_cast<long long*>(b->h_stage);
  int* h_off = reinterpret_cast<int*>(b->h_stage + o_off);
  int* h_warm = reinterpret_cast<int*>(b->h_stage + o_warm);
  int* h_large = reinterpret_cast<int*>(b->h_stage + o_large);
  int nlarge = 0, maxn = 0;
  BatchCost cost{};
  size_t wanted = 0;   // pairs of all tables
  for (int c = 0; c < n_clusters; ++c) {
    h_off[c] = site_offsets[c];
    h_warm[c] = warm_start ? (warm_start[c] != 0) : 0;
    const int nc = site_offsets[c + 1] - site_offsets[c];
    h_coef[c] = -1;
    if (nc <= kClSmall) {
      ++cost.ns;
      cost.cs += cluster_cost(nc);
      continue;
    }
    ++cost.nl;
    cost.cl += cluster_cost(nc);
    cost.ml = std::max(cost.ml, cluster_cost(nc));
    h_large[nlarge++] = c;
    maxn = std::max(maxn, nc);
    const size_t np = std::min(nc, kClMaxPol);
    if ((wanted + np * np) * pair_bytes <= kClTableBytes) wanted += np * np;
  }
  h_off[n_clusters] = site_offsets[n_clusters];
  const sibfa_status grown = grow_table(b, wanted * pair_bytes);
  if (grown != SIBFA_OK) return grown;
  bool bare = false;   // large clusters without a table
  size_t pairs = 0;
  for (int k = 0; k < nlarge; ++k) {
    const int c = h_large[k];
    const size_t np = std::min(site_offsets[c + 1] - site_offsets[c], kClMaxPol);
    if ((pairs + np * np) * pair_bytes <= std::min(b->table_bytes, kClTableBytes)) {
      h_coef[c] = (long long)pairs;
      pairs += np * np;
    } else {
      bare = true;
    }
  }
  if (pairs > 0) {
    a.coef = static_cast<double2*>(b->table);
    a.coef32 = mix ? reinterpret_cast<float2*>(a.coef + pairs) : nullptr;
  } else {
    a.coef_off = nullptr;   // none needed, or no memory for them
  }
  BHIP(hipMemcpyAsync(b->scratch, b->h_stage, nlarge > 0 ? need : o_warm + n_clusters * sizeof(int),
                      hipMemcpyHostToDevice, b->stream));
  BHIP(hipEventRecord(b->staged, b->stream));
  b->staged_pending = true;
  a.nclusters = n_clusters;
  a.nsites = (int)n;
  a.xyz = xyz;
  a.mol = mol;
  a.q = q;
  a.dip = dip;
  a.quad = quad;
  a.alpha = alpha;
  a.thole = thole;
  a.thole_a = params->thole_a;
  a.tol = params->tol_debye;
  a.max_iter = params->max_iter;
  a.mu = mu;
  a.forces = forces;
  a.e_pol = e_pol;
  a.e_elec = e_elec;
  a.iters = iterations;
  a.rms = rms_debye;
  a.status = status;
  a.apart = nullptr;   // decided here
  BatchPlan p;
  p.gs = std::min(n_clusters, 16384);
  p.apart = cost.ns > 0 && small_apart(cost);
  p.beside = cost.ns > 0 && !p.apart;
  p.large = nlarge;
  p.gx = std::min(nlarge, 16384);
  p.bare = bare;
  p.tiles = (maxn + kClTile - 1) / kClTile;
  if (mix) launch_batch<float>(a, p, b->stream);
  else launch_batch<double>(a, p, b->stream);
  BHIP(hipGetLastError());
  return SIBFA_OK;
}

}  // extern "C"

namespace {

constexpr int kNaMaxDevices = 64;
std::mutex g_na_mu;
void* g_na_ptr[kNaMaxDevices] = {};

// Device address of `scratch` on `device` (which must be current), looked
// up once per device.  In host code the array's name is only a stand-in
// for the symbol: kernels get this address.
sibfa_status noalloc_scratch(int device, void** out) {
  std::lock_guard<std::mutex> lock(g_na_mu);
  if (!g_na_ptr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SIBFA_E_DEVICE;
    g_na_ptr[device] = p;
  }
  *out = g_na_ptr[device];
  return SIBFA_OK;
}

}  // namespace

extern "C" sibfa_status sibfa_batch_clusters_noalloc(
    int device, void* hip_stream, int n_clusters, int n_sites, const int* site_offsets,
    const int* warm_start, const double* xyz, const int32_t* mol, const double* q,
    const double* dip, const double* quad, const double* alpha, const double* thole,
    const sibfa_params* params, double* mu, double* forces, double* e_pol, double* e_elec,
    int* iterations, double* rms_debye, int* status) {
  if (n_clusters < 1 || n_clusters > SIBFA_BATCH_NOALLOC_MAX_CLUSTERS || n_sites < 1 ||
      n_sites > SIBFA_BATCH_NOALLOC_MAX_SITES)
    return SIBFA_E_ARG;
  if (!site_offsets || !xyz || !mol || !q || !dip || !quad || !alpha || !params || !mu ||
      !e_pol || !e_elec || !iterations || !rms_debye || !status)
    return SIBFA_E_ARG;
  if (!(params->tol_debye > 0.0) || params->max_iter < 1 || !(params->thole_a > 0.0) ||
      (params->precision != SIBFA_FP64 && params->precision != SIBFA_MIXED))
    return SIBFA_E_ARG;
  if (device < 0 || device >= kNaMaxDevices) return SIBFA_E_DEVICE;
  if (hipSetDevice(device) != hipSuccess) return SIBFA_E_DEVICE;
  // the layout of carve() must fit the static array
  if (carve(nullptr, kNaSites, kNaClusters, nullptr) > kNaBytes) return SIBFA_E_DEVICE;
  void* base = nullptr;
  if (noalloc_scratch(device, &base) != SIBFA_OK) return SIBFA_E_DEVICE;
  ClusterArgs a{};
  carve(static_cast<char*>(base), kNaSites, kNaClusters, &a);
  a.off = site_offsets;   // the caller's device arrays, checked per cluster
  a.warm = warm_start;
  // Sizes are known on the device only: k_cl_prep lists the large clusters, of
  // which at most gx fit n_sites (ranges that overlap, which could be more,
  // wait their turn).  Small clusters look in both places where they may run.
  BatchPlan p;
  p.gs = n_clusters;
  p.apart = true;
  p.large = n_sites > kClSmall ? n_clusters : 0;
  p.beside = p.large > 0;
  p.gx = std::max(1, std::min(n_clusters, n_sites / (kClSmall + 1)));
  p.bare = true;
  p.tiles = std::min(kClMaxSites / kClTile, 8);
  a.list = p.large > 0 ? const_cast<int*>(a.large) : nullptr;
  if (p.large == 0) a.apart = nullptr;
  a.coef_off = nullptr;   // no room for tables
  a.nclusters = n_clusters;
  a.nsites = n_sites;
  a.xyz = xyz;
  a.mol = mol;
  a.q = q;
  a.dip = dip;
  a.quad = quad;
  a.alpha = alpha;
  a.thole = thole;
  a.thole_a = params->thole_a;
  a.tol = params->tol_debye;
  a.max_iter = params->max_iter;
  a.mu = mu;
  a.forces = forces;
  a.e_pol = e_pol;
  a.e_elec = e_elec;
  a.iters = iterations;
  a.rms = rms_debye;
  a.status = status;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  if (params->precision == SIBFA_MIXED) launch_batch<float>(a, p, st);
  else launch_batch<double>(a, p, st);
  return hipGetLastError() == hipSuccess ? SIBFA_OK : SIBFA_E_DEVICE;
}
