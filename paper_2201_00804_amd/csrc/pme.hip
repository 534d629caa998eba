// Smooth PME: B-spline spreading of multipoles onto the charge grid and
// gathering of potential derivatives (Essmann et al. 1995, the SPME method
// the paper uses for multipoles and polarization).
//
// With u_a = K_a r_a / L_a and W(k) = prod_a M_p(u_a - k_a), a site adds
//   q W + d.grad W + 1/3 Theta:grad grad W
// to grid point k (gradients with respect to the site position, so a
// derivative along a carries K_a/L_a).  After the convolution the grid holds
// the potential phi(k); a site's potential derivatives are sums of phi(k)
// times derivatives of W.  Grid layout: x fastest, [K2][K1][K0].
// Spreading accumulates in LDS per grid brick (see below); gathering reads
// p^3 points per site in p*p rows of p consecutive addresses.
#include "common.h"
#include "kernels.h"

namespace sibfa {

// ------------------------------------------------------------ spreading
// Sites are binned by home brick, the brick of B^3 grid points (B <= 8, per
// axis; no brick has fewer than p - 1 points along an axis) holding their base
// index b.  A site touches points b - t, t = 0..p-1, so all contributions of a brick's sites fall in the brick extended by p - 1
// points towards lower indices: its tile, (B + p - 1)^3 points.
//
//  k_spread_tile : one workgroup per brick spreads its own sites into the
//                  tile (every site is evaluated once) and stores the tile;
//  fold          : every grid point sums the tiles that cover it -- its own
//                  brick's and, along each axis where it lies within p - 1
//                  points of the next brick, that brick's -- in a fixed
//                  order.  No global atomics, no clearing, deterministic.
//                  k_spread_fold writes the real grid Q the convolution
//                  starts from, or its first pass sums the tiles itself.

// Sites come in cell-sorted order, so a wavefront's sites fall in a few
// bricks: one counter atomic per run of equal bricks.  One pass bins all
// sites and, among them, the polarizable ones (slot: brick, slot in the
// brick's list of all sites and in that of its polarizable sites).
__global__ void k_brick_bin(SysView s, PmeView pm, int3* slot, int* count_all, int* count_pol) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool act = i < s.n;
  int b = 0, pi = -1;
  if (act) {
    const double4 p = s.sp[i];
    pi = s.polidx[i];
    const double x[3] = {p.x, p.y, p.z};
    int h[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double fr;
      h[a] = brick_of(pm, a, grid_base(x[a], pm.scale[a], pm.K[a], &fr));
    }
    b = h[0] + pm.nb[0] * (h[1] + pm.nb[1] * h[2]);
  }
  const int sa = wave_atomic_inc(count_all, b, act);
  const int sp = wave_atomic_inc(count_pol, b, act && pi >= 0);
  if (act) slot[i] = make_int3(b, sa, sp);
}

__global__ void k_brick_scatter(SysView s, const int3* slot, const int* start_all, int* order_all,
                                const int* start_pol, int* order_pol) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= s.n) return;
  const int3 q = slot[i];
  order_all[start_all[q.x] + q.y] = i;
  const int pi = s.polidx[i];
  if (pi >= 0) order_pol[start_pol[q.x] + q.z] = pi;
}

void launch_brick_bin(const SysView& s, const PmeView& pm, int3* slot, int* count_all,
                      int* count_pol, hipStream_t st) {
  hipLaunchKernelGGL(k_brick_bin, dim3((s.n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, s, pm,
                     slot, count_all, count_pol);
}

void launch_brick_scatter(const SysView& s, const int3* slot, const int* start_all, int* order_all,
                          const int* start_pol, int* order_pol, hipStream_t st) {
  hipLaunchKernelGGL(k_brick_scatter, dim3((s.n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, s,
                     slot, start_all, order_all, start_pol, order_pol);
}

template <typename R>
__device__ __forceinline__ R* grid_out(const PmeView& pm);
template <>
__device__ __forceinline__ double* grid_out<double>(const PmeView& pm) { return pm.Q; }
template <>
__device__ __forceinline__ float* grid_out<float>(const PmeView& pm) { return pm.Q32; }
template <typename R>
__device__ __forceinline__ R* tile_buf(const PmeView& pm);
template <>
__device__ __forceinline__ double* tile_buf<double>(const PmeView& pm) { return pm.tiles; }
template <>
__device__ __forceinline__ float* tile_buf<float>(const PmeView& pm) { return pm.tiles32; }

// B-spline weights of order P at offset w (derivatives up to ND <= 2) with
// every rounding written out (explicit fused multiply-adds, contraction
// off), so that the FP32 grid keeps its bits whatever code surrounds this:
// the recursion of bspline_weights, a first derivative fused with the
// scaling of its level.
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <typename R, int P, int ND>
__device__ __forceinline__ void spread_weights(R w, R th[ND + 1][P]) {
#pragma clang fp contract(off)
  R lev[P][P], num[P][P];   // lev[k][t] = num / k = M_{k+1}(w + t)
  lev[0][0] = R(1);
#pragma unroll
  for (int t = 1; t < P; ++t) lev[0][t] = R(0);
#pragma unroll
  for (int k = 1; k < P; ++k) {
    const R inv = R(1) / R(k);
#pragma unroll
    for (int t = P - 1; t >= 0; --t) {
      const R u = w + R(t);
      const R a = t <= k - 1 ? lev[k - 1][t] : R(0);
      const R b = t >= 1 && t - 1 <= k - 1 ? lev[k - 1][t - 1] : R(0);
      num[k][t] = fma_(u, a, (R(k + 1) - u) * b);
      lev[k][t] = num[k][t] * inv;
    }
  }
#pragma unroll
  for (int t = 0; t < P; ++t) {
    th[0][t] = lev[P - 1][t];
    if (ND >= 1)
      th[ND >= 1 ? 1 : 0][t] =
          t == 0 ? lev[P - 2][0] : fma_(R(1) / R(P - 2), num[P - 2][t], -lev[P - 2][t - 1]);
    if (ND >= 2) {
      const R b = t >= 1 ? lev[P - 3][t - 1] : R(0), c = t >= 2 ? lev[P - 3][t - 2] : R(0);
      th[ND >= 2 ? 2 : 0][t] = fma_(b, R(-2), lev[P - 3][t]) + c;
    }
  }
}

// FULL: multipoles (q, d [+ mu], Theta) of all sites; otherwise the dipoles
// of the polarizable sites.
//
// One workgroup of two waves per brick, the tile in LDS.  The second wave
// stages the brick's sites in chunks (amplitudes, and the P weights and
// their derivatives per axis, three lanes per site); meanwhile the first
// walks the chunk before, site by site in order, and adds each site's p^3
// points to the tile, one point per lane (two rounds at p = 5): a read, the
// three-axis product and a write per point, no atomics: a wave's LDS accesses
// are carried out in order, and wave_sync() keeps the compiler to it.  Bound by instruction issue of the first wave,
// about 36 per site and one every five cycles.  A thread per tile column
// instead, its z values in registers, spent 5% of its multiply-adds on
// points inside the site's support and 70 instructions of three waves per
// site; splitting the tile's planes over four waves leaves each of them
// most of the sites.  Dipole spread, thread per column -> this: 28 -> 16 us
// at 4,096 waters (FP32), 81 -> 40 us at 32,000 (FP64, beside the matvec);
// all multipoles 53 -> 32 us in the 27 bricks of 18^3 points that 216 waters
// had (13 us in the 64 they have now).
// The brick lists are sorted by site index when they are built and one wave
// adds them in that order, so the tile sums -- and the grid -- are
// reproducible bit for bit.
constexpr int kSpreadChunk = 21;   // sites per chunk: three lanes each of one wave

template <bool FULL>
struct SpreadShape {
  static constexpr int ND = FULL ? 2 : 1;    // highest derivative order
  static constexpr int NK = FULL ? 4 : 2;    // weights kept per point and axis (padded)
  static constexpr int NA = FULL ? 12 : 4;   // amplitudes per site (padded)
};

template <typename R, int P, bool FULL>
struct SpreadChunk {
  using Sh = SpreadShape<FULL>;
  R wt[kSpreadChunk][3][P][Sh::NK];
  R amp[kSpreadChunk][Sh::NA];
  int top[kSpreadChunk];   // tile index of the site's highest point
};

// Site j of a chunk by the lane 3 j + ax of axis ax: idx its index, o the
// axis' brick origin, T0 and T1 the tile's extents.
template <typename R, int P, bool FULL>
__device__ __forceinline__ void stage_site(const SysView& s, const PmeView& pm, const double4* vec,
                                           SpreadChunk<R, P, FULL>& c, int j, int ax, int idx,
                                           int o, int T0, int T1) {
#pragma clang fp contract(off)
  using Sh = SpreadShape<FULL>;
  constexpr int ND = Sh::ND, NA = Sh::NA;
  const double4 p = FULL ? s.sp[idx] : s.pp[idx];
  const double xa = ax == 0 ? p.x : (ax == 1 ? p.y : p.z);
  double fr;
  const int base = grid_base(xa, pm.scale[ax], pm.K[ax], &fr);
  R th[ND + 1][P];
  spread_weights<R, P, ND>((R)fr, th);
  const int top = base - o + P - 1;
  const int ty = __shfl(top, 3 * j + 1, 64), tz = __shfl(top, 3 * j + 2, 64);
#pragma unroll
  for (int t = 0; t < P; ++t)
#pragma unroll
    for (int k = 0; k <= ND; ++k) c.wt[j][ax][t][k] = th[k][t];
  if (ax != 0) return;
  c.top[j] = (tz * T1 + ty) * T0 + top;
  const R sc[3] = {(R)pm.scale[0], (R)pm.scale[1], (R)pm.scale[2]};
  R* A = c.amp[j];
  if (FULL) {
    const double4 d4 = s.sd[idx], t4 = s.sth[idx];
    const double2 t2 = s.sth2[idx];
    double ddx = d4.x, ddy = d4.y, ddz = d4.z;
    if (vec) {
      const double4 m = vec[idx];
      ddx += m.x; ddy += m.y; ddz += m.z;
    }
    const R third = R(1.0 / 3.0);
    A[0] = (R)p.w;
    A[1] = (R)ddx * sc[0];
    A[2] = (R)ddy * sc[1];
    A[3] = (R)ddz * sc[2];
    A[4 % NA] = (R)t4.x * sc[0] * sc[0] * third;
    A[5 % NA] = (R)t4.w * sc[1] * sc[1] * third;
    A[6 % NA] = (R)t2.y * sc[2] * sc[2] * third;
    A[7 % NA] = R(2) * third * (R)t4.y * sc[0] * sc[1];
    A[8 % NA] = R(2) * third * (R)t4.z * sc[0] * sc[2];
    A[9 % NA] = R(2) * third * (R)t2.x * sc[1] * sc[2];
  } else {
    const double4 pv = vec[idx];
    A[0] = (R)pv.x * sc[0];
    A[1] = (R)pv.y * sc[1];
    A[2] = (R)pv.z * sc[2];
  }
}

template <typename R, int P, bool FULL>
__global__ __launch_bounds__(128) void k_spread_tile(SysView s, PmeView pm, const double4* vec) {
#pragma clang fp contract(off)
  if (stopped(pm.stop)) return;
  using Sh = SpreadShape<FULL>;
  constexpr int NK = Sh::NK, NA = Sh::NA, CH = kSpreadChunk;
  constexpr int TM = kBrick + P - 1, P3 = P * P * P, NR = (P3 + 63) / 64;
  __shared__ __align__(16) R tile[TM * TM * TM];
  __shared__ __align__(16) SpreadChunk<R, P, FULL> chunk[2];
  const int tid = threadIdx.x, lane = tid & 63;
  const bool stager = tid >= 64;
  const int b = blockIdx.x;
  const int* start = FULL ? pm.bstart_all : pm.bstart_pol;
  const int* order = FULL ? pm.border_all : pm.border_pol;
  const int s0 = start[b], total = start[b + 1] - s0;
  const int T0 = pm.Bb[0] + P - 1, T1 = pm.Bb[1] + P - 1, T2 = pm.Bb[2] + P - 1;
  const int nb0 = pm.nb[0], nb1 = pm.nb[1], size = T0 * T1 * T2;
  // the stager's site and axis; the spreader's points: offsets from a site's
  // highest one and places of their weights (a lane past the support repeats
  // the last point: the same value written twice)
  const int sj = lane / 3, ax = lane - 3 * sj;
  const int o = brick_start(pm, ax, ax == 0 ? b % nb0 : ax == 1 ? (b / nb0) % nb1
                                                                : b / (nb0 * nb1));
  int dx[NR], dy[NR], dz[NR], off[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = min(lane + 64 * r, P3 - 1);
    dx[r] = q % P;
    dy[r] = q / P % P;
    dz[r] = q / (P * P);
    off[r] = (dz[r] * T1 + dy[r]) * T0 + dx[r];
  }
  if (stager) {
    if (sj < min(CH, total))
      stage_site<R, P, FULL>(s, pm, vec, chunk[0], sj, ax, order[s0 + sj], o, T0, T1);
  } else {
    for (int i = lane; i < size; i += 64) tile[i] = R(0);
  }
  int buf = 0;
  for (int c0 = 0; c0 < total; c0 += CH, buf ^= 1) {
    __syncthreads();   // chunk `buf` is staged, the other one is spread
    const int n = min(CH, total - c0);
    if (stager) {
      const int e = c0 + CH + sj;
      if (sj < CH && e < total)
        stage_site<R, P, FULL>(s, pm, vec, chunk[buf ^ 1], sj, ax, order[s0 + e], o, T0,
                               T1);
      continue;
    }
    const SpreadChunk<R, P, FULL>& c = chunk[buf];
    auto value = [&](int j, R v[NR]) {
#pragma clang fp contract(off)
      const R* A = c.amp[j];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const R* X = c.wt[j][0][dx[r]];
        const R* Y = c.wt[j][1][dy[r]];
        const R* Z = c.wt[j][2][dz[r]];
        if (FULL) {
          const R U0 = fma_(X[2 % NK] * A[4 % NA], Y[0],
                            fma_(X[0], fma_(A[5 % NA], Y[2 % NK], fma_(A[0], Y[0], A[2] * Y[1])),
                                 X[1] * fma_(A[1], Y[0], A[7 % NA] * Y[1])));
          const R U1 = fma_(X[0], fma_(A[3], Y[0], A[9 % NA] * Y[1]), X[1] * A[8 % NA] * Y[0]);
          const R U2 = X[0] * A[6 % NA] * Y[0];
          v[r] = fma_(U2, Z[2 % NK], fma_(U0, Z[0], U1 * Z[1]));
        } else {
          const R U0 = fma_(A[0] * X[1], Y[0], A[1] * X[0] * Y[1]);
          const R U1 = A[2] * X[0] * Y[0];
          v[r] = fma_(U0, Z[0], U1 * Z[1]);
        }
      }
    };
    // other lanes wrote these points for the site before: its writes come first
    auto add = [&](int base, const R v[NR]) {
      wave_sync();
      R t[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) t[r] = tile[base - off[r]];
#pragma unroll
      for (int r = 0; r < NR; ++r) tile[base - off[r]] = t[r] + v[r];
    };
    // two sites' weights are read before the first touches the tile
    int j = 0;
    for (; j + 1 < n; j += 2) {
      R v0[NR], v1[NR];
      const int b0 = c.top[j], b1 = c.top[j + 1];
      value(j, v0);
      value(j + 1, v1);
      add(b0, v0);
      add(b1, v1);
    }
    if (j < n) {
      R v[NR];
      value(j, v);
      add(c.top[j], v);
    }
  }
  __syncthreads();
  R* out = tile_buf<R>(pm) + (size_t)b * pm.tile_size;
  for (int i = tid; i < size; i += 128) out[i] = tile[i];
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_spread_fold(PmeView pm) {
  if (stopped(pm.stop)) return;
  const int K0 = pm.K[0], K1 = pm.K[1], K2 = pm.K[2];
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)K0 * K1 * K2) return;
  grid_out<R>(pm)[idx] = fold_point<R>(pm, (int)(idx % K0), (int)((idx / K0) % K1),
                                       (int)(idx / ((size_t)K0 * K1)));
}

void launch_spread_fold(const PmeView& pm, bool mixed, hipStream_t st) {
  const size_t npts = (size_t)pm.K[0] * pm.K[1] * pm.K[2];
  const dim3 g((unsigned)((npts + kBlock - 1) / kBlock)), b(kBlock);
  if (mixed) hipLaunchKernelGGL(k_spread_fold<float>, g, b, 0, st, pm);
  else hipLaunchKernelGGL(k_spread_fold<double>, g, b, 0, st, pm);
}

// ------------------------------------------------------------ gathering
template <typename R, int P>
__global__ __launch_bounds__(kBlock) void k_gather_field(SysView s, PmeView pm, double4* E0) {
  const int pi = blockIdx.x * blockDim.x + threadIdx.x;
  if (pi >= s.npol) return;
  const double4 x = s.pp[pi];
  int base[3];
  R th[3][2][P];
  site_splines<R, P, 1>(pm, x.x, x.y, x.z, base, th);
  double g[3] = {0.0, 0.0, 0.0};
  for (int tz = 0; tz < P; ++tz) {
    GridRow<R, P> row[P];
    grid_rows<R, P>(pm, base, tz, row);
#pragma unroll
    for (int ty = 0; ty < P; ++ty) {
      R s0 = 0, s1 = 0;
#pragma unroll
      for (int tx = 0; tx < P; ++tx) {
        const R v = row[ty][tx];
        s0 += v * th[0][0][tx];
        s1 += v * th[0][1][tx];
      }
      g[0] += (double)(s1 * th[1][0][ty] * th[2][0][tz]);
      g[1] += (double)(s0 * th[1][1][ty] * th[2][0][tz]);
      g[2] += (double)(s0 * th[1][0][ty] * th[2][1][tz]);
    }
  }
  double4 e = E0[pi];
  e.x -= g[0] * pm.scale[0];
  e.y -= g[1] * pm.scale[1];
  e.z -= g[2] * pm.scale[2];
  E0[pi] = e;
}

// index of the (kx, ky, kz) derivative, kx + ky + kz <= 3
__host__ __device__ constexpr int didx(int kx, int ky, int kz) {
  return kx + 4 * (ky + 4 * kz);
}

// Reciprocal forces of the combined density at every site.  VIR: also the
// site terms of the reciprocal virial, sum_j [d'_jb d_a phi(r_j) +
// 2/3 Theta_jbc d_a d_c phi(r_j)] with d' = d + mu (block partials, slots
// S_VRG, row-major).
template <typename R, int P, bool VIR>
__global__ __launch_bounds__(kBlock) void k_gather_force(SysView s, PmeView pm, Reduce red,
                                                         const double4* mu, const double4* Freal,
                                                         const int* perm, double* out,
                                                         double4* FS, double* GS, bool self) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  double W[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (i < s.n) {
    const double4 p = s.sp[i], d4 = s.sd[i], t4 = s.sth[i];
    const double2 t2 = s.sth2[i];
    const double4 m = mu[i];
    int base[3];
    R th[3][4][P];
    site_splines<R, P, 3>(pm, p.x, p.y, p.z, base, th);
    double D[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) D[k] = 0.0;
#pragma unroll
    for (int tz = 0; tz < P; ++tz) {
      GridRow<R, P> row[P];
      grid_rows<R, P>(pm, base, tz, row);
#pragma unroll
      for (int ty = 0; ty < P; ++ty) {
        R sx[4] = {0, 0, 0, 0};
#pragma unroll
        for (int tx = 0; tx < P; ++tx) {
          const R v = row[ty][tx];
#pragma unroll
          for (int k = 0; k < 4; ++k) sx[k] += v * th[0][k][tx];
        }
#pragma unroll
        for (int kz = 0; kz <= 3; ++kz)
#pragma unroll
          for (int ky = 0; ky <= 3 - kz; ++ky) {
            const R yz = th[1][ky][ty] * th[2][kz][tz];
#pragma unroll
            for (int kx = 0; kx <= 3 - ky - kz; ++kx) D[didx(kx, ky, kz)] += (double)(sx[kx] * yz);
          }
      }
    }
    const double sc[3] = {pm.scale[0], pm.scale[1], pm.scale[2]};
    auto der = [&](int a, int b, int c) -> double {   // b, c = -1 for lower order
      int k[3] = {0, 0, 0};
      double f = sc[a];
      k[a]++;
      if (b >= 0) { k[b]++; f *= sc[b]; }
      if (c >= 0) { k[c]++; f *= sc[c]; }
      return D[didx(k[0], k[1], k[2])] * f;
    };
    const double q = p.w;
    const double dd[3] = {d4.x + m.x, d4.y + m.y, d4.z + m.z};
    const double T[3][3] = {{t4.x, t4.y, t4.z}, {t4.y, t4.w, t2.x}, {t4.z, t2.x, t2.y}};
    const double4 fr = Freal[i];
    const double frr[3] = {fr.x, fr.y, fr.z};
    const int c = perm[i];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double f = q * der(a, -1, -1);
      for (int b = 0; b < 3; ++b) {
        f += dd[b] * der(a, b, -1);
        for (int cc = 0; cc < 3; ++cc) f += T[b][cc] * der(a, b, cc) * (1.0 / 3.0);
      }
      out[3 * (size_t)c + a] = kCoulomb * (frr[a] - f);
    }
    if (FS) {
      // site field E = -grad phi and gradient -grad grad phi, plus the self
      // terms: 4 b^3/(3 sqrt pi) (d + mu) and 16 b^5/(15 sqrt pi) Theta
      // (the latter 3x the quadrupole self derivative, as the field
      // gradient enters the quadrupole energy with 1/3)
      const double b = pm.beta, b3 = b * b * b;
      const double sf = self ? 4.0 * b3 / (3.0 * kSqrtPi) : 0.0;
      const double st = self ? 16.0 * b3 * b * b / (15.0 * kSqrtPi) : 0.0;
      double4 e = FS[i];
      e.x += sf * dd[0] - der(0, -1, -1);
      e.y += sf * dd[1] - der(1, -1, -1);
      e.z += sf * dd[2] - der(2, -1, -1);
      FS[i] = e;
      const int ia[6] = {0, 0, 0, 1, 1, 2}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
      for (int k = 0; k < 6; ++k)
        GS[6 * (size_t)i + k] += st * T[ia[k]][ib[k]] - der(ia[k], ib[k], -1);
    }
    if (VIR) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double da = der(a, -1, -1);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          double w = dd[b] * da;
#pragma unroll
          for (int cc = 0; cc < 3; ++cc) w += (2.0 / 3.0) * T[b][cc] * der(a, cc, -1);
          W[3 * a + b] = w;
        }
      }
    }
  }
  if (VIR)
#pragma unroll
    for (int k = 0; k < 9; ++k) block_partial(W[k], red, S_VRG + k);
}

// ------------------------------------------------------------ launchers
template <int P, bool FULL>
static void spread_p(const PmeView& pm, const SysView& s, const double4* vec, bool mixed,
                     hipStream_t st) {
  const dim3 g(pm.nb[0] * pm.nb[1] * pm.nb[2]), bt(128);
  if (mixed) hipLaunchKernelGGL((k_spread_tile<float, P, FULL>), g, bt, 0, st, s, pm, vec);
  else hipLaunchKernelGGL((k_spread_tile<double, P, FULL>), g, bt, 0, st, s, pm, vec);
}

template <bool FULL>
static void spread(const PmeView& pm, const SysView& s, const double4* vec, bool mixed,
                   hipStream_t st) {
  switch (pm.order) {
    case 4: spread_p<4, FULL>(pm, s, vec, mixed, st); break;
    case 6: spread_p<6, FULL>(pm, s, vec, mixed, st); break;
    default: spread_p<5, FULL>(pm, s, vec, mixed, st); break;
  }
}

void launch_spread_mult(const SysView& s, const PmeView& pm, const double4* mu, bool mixed,
                        hipStream_t st) {
  spread<true>(pm, s, mu, mixed, st);
}

void launch_spread_dip(const SysView& s, const PmeView& pm, const double4* p, bool mixed,
                       hipStream_t st) {
  spread<false>(pm, s, p, mixed, st);
}

// Sites per workgroup of the gathers: one wavefront up to 65,536 sites (256
// workgroups of four), so that few sites still spread over the CUs, whose
// texture paths bound them.  Forces with four / one (FP64): 4,860 to 14,400 sites
// 8.9 / 7.2 us, 46,305 9.6 / 9.0, 60,835 10.4 / 12.1; from 69,000 on the same.
static dim3 gather_block(int n) { return dim3(n <= 256 * kBlock ? 64 : kBlock); }

template <int P>
static void gather_field_p(const SysView& s, const PmeView& pm, double4* E0, bool mixed,
                           hipStream_t st) {
  if (s.npol <= 0) return;
  const dim3 b = gather_block(s.npol), g((s.npol + b.x - 1) / b.x);
  if (mixed) hipLaunchKernelGGL((k_gather_field<float, P>), g, b, 0, st, s, pm, E0);
  else hipLaunchKernelGGL((k_gather_field<double, P>), g, b, 0, st, s, pm, E0);
}

void launch_gather_field(const SysView& s, const PmeView& pm, double4* E0, bool mixed,
                         hipStream_t st) {
  switch (pm.order) {
    case 4: gather_field_p<4>(s, pm, E0, mixed, st); break;
    case 6: gather_field_p<6>(s, pm, E0, mixed, st); break;
    default: gather_field_p<5>(s, pm, E0, mixed, st); break;
  }
}

template <int P, bool VIR>
static void gather_force_pv(const SysView& s, const PmeView& pm, Reduce& red, const double4* mu,
                            const double4* Freal, const int* perm, double* out, bool mixed,
                            hipStream_t st, double4* FS, double* GS, bool self) {
  const dim3 b = gather_block(s.n), g((s.n + b.x - 1) / b.x);
  if (mixed)
    hipLaunchKernelGGL((k_gather_force<float, P, VIR>), g, b, 0, st, s, pm, red, mu, Freal, perm,
                       out, FS, GS, self);
  else
    hipLaunchKernelGGL((k_gather_force<double, P, VIR>), g, b, 0, st, s, pm, red, mu, Freal, perm,
                       out, FS, GS, self);
  if (VIR)
    for (int k = 0; k < 9; ++k) red.nparts[S_VRG + k] = (int)g.x;
}

template <int P>
static void gather_force_p(const SysView& s, const PmeView& pm, Reduce& red, const double4* mu,
                           const double4* Freal, const int* perm, double* out, bool mixed,
                           bool vir, hipStream_t st, double4* FS, double* GS, bool self) {
  if (vir) gather_force_pv<P, true>(s, pm, red, mu, Freal, perm, out, mixed, st, FS, GS, self);
  else gather_force_pv<P, false>(s, pm, red, mu, Freal, perm, out, mixed, st, FS, GS, self);
}

void launch_gather_force(const SysView& s, const PmeView& pm, Reduce& red, const double4* mu,
                         const double4* Freal, const int* perm, double* out, bool mixed,
                         bool virial, hipStream_t st, double4* FS, double* GS, bool self) {
  switch (pm.order) {
    case 4: gather_force_p<4>(s, pm, red, mu, Freal, perm, out, mixed, virial, st, FS, GS, self); break;
    case 6: gather_force_p<6>(s, pm, red, mu, Freal, perm, out, mixed, virial, st, FS, GS, self); break;
    default: gather_force_p<5>(s, pm, red, mu, Freal, perm, out, mixed, virial, st, FS, GS, self); break;
  }
}

}  // namespace sibfa
