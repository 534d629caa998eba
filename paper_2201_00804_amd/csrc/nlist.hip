// Cell binning, deterministic cell sort, per-site records and real-space
// neighbour lists.
//
// Sites are binned into cells of edge >= cutoff/2 (a 5x5x5 cell stencil
// then covers the cutoff sphere), counting-sorted by cell, and each cell's
// segment is sorted by caller index so that the order -- and with it every
// summation order downstream -- is reproducible (a cluster is one cell, in
// caller order).  The neighbour-list kernel runs one or more wavefronts per
// cell: 64 candidate sites are loaded per step and tested against the
// wavefront's sites; hits are compacted with lane masks so list order is
// deterministic too.  Four ELL lists are produced:
//   all   intermolecular site pairs within the cutoff (E, E_elec, forces)
//   in    same-molecule site pairs (excluded or damped, always present)
//   pol   intermolecular polarizable pairs within the cutoff (T)
//   ipol  same-molecule polarizable pairs (T, Thole-damped)
#include <algorithm>
#include <initializer_list>
#include <utility>

#include "common.h"
#include "nlist.h"

namespace sibfa {

// ------------------------------------------------------------ fill / scan
template <typename T>
__global__ void k_fill(T* p, T v, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

static int fill_blocks(size_t n) {
  size_t b = (n + kBlock - 1) / kBlock;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

void launch_fill_int(int* p, int v, size_t n, hipStream_t s) {
  if (n) hipLaunchKernelGGL(k_fill<int>, dim3(fill_blocks(n)), dim3(kBlock), 0, s, p, v, n);
}
void launch_fill_double(double* p, double v, size_t n, hipStream_t s) {
  if (n) hipLaunchKernelGGL(k_fill<double>, dim3(fill_blocks(n)), dim3(kBlock), 0, s, p, v, n);
}
void launch_fill_float(float* p, float v, size_t n, hipStream_t s) {
  if (n) hipLaunchKernelGGL(k_fill<float>, dim3(fill_blocks(n)), dim3(kBlock), 0, s, p, v, n);
}

// Several int buffers set to one value in a single launch.
__global__ void k_fill_ints(FillList f) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (int k = 0; k < f.n; ++k)
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < f.cnt[k]; i += stride)
      f.p[k][i] = f.v;
}

void launch_fill_ints(std::initializer_list<std::pair<int*, size_t>> bufs, int v, hipStream_t s) {
  FillList f{};
  size_t mx = 0;
  for (const auto& b : bufs) {
    if (f.n == kFillMax) {   // more than one launch's worth
      hipLaunchKernelGGL(k_fill_ints, dim3(fill_blocks(mx)), dim3(kBlock), 0, s, f);
      f.n = 0;
      mx = 0;
    }
    f.p[f.n] = b.first;
    f.cnt[f.n] = b.second;
    ++f.n;
    mx = std::max(mx, b.second);
  }
  f.v = v;
  if (f.n && mx) hipLaunchKernelGGL(k_fill_ints, dim3(fill_blocks(mx)), dim3(kBlock), 0, s, f);
}

constexpr int kScanTile = 4 * kBlock;   // elements per block

__device__ int block_exclusive_scan(int v, int* total) {
  __shared__ int wsum[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int x = v;
  for (int off = 1; off < 64; off <<= 1) {
    int y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  int base = 0, tot = 0;
  for (int w = 0; w < kBlock / 64; ++w) {
    if (w < wid) base += wsum[w];
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return base + x - v;
}

__global__ void k_scan_tiles(const int* in, int* out, int n, int* tile_sums) {
  const int base = blockIdx.x * kScanTile + threadIdx.x * 4;
  int v[4], s = 0;
  for (int k = 0; k < 4; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0;
    s += v[k];
  }
  int total;
  int ex = block_exclusive_scan(s, &total);
  for (int k = 0; k < 4; ++k) {
    if (base + k < n) out[base + k] = ex;
    ex += v[k];
  }
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

__global__ void k_scan_add(int* out, int n, const int* tile_offsets) {
  const int base = blockIdx.x * kScanTile + threadIdx.x * 4;
  const int add = tile_offsets[blockIdx.x];
  for (int k = 0; k < 4; ++k)
    if (base + k < n) out[base + k] += add;
}

// Exclusive scan of up to kScanSingleMax (16,384) values by one 1,024-thread
// workgroup: tiles of 4,096 values in order, each scanned in registers and
// across the wavefronts, with the running total carried to the next tile.
// One launch instead of the three of the multi-block form.
constexpr int kScanBig = 1024;
constexpr int kScanSingleMax = 4 * 4 * kScanBig;   // larger scans: the multi-block form is faster
struct ScanArgs {
  const int* in[2];
  int* out[2];
  int n;
};
__global__ __launch_bounds__(kScanBig) void k_scan_single(ScanArgs a) {
  const int* in = a.in[blockIdx.x];
  int* out = a.out[blockIdx.x];
  const int n = a.n;
  __shared__ int wsum[kScanBig / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int carry = 0;
  for (int t0 = 0; t0 < n; t0 += 4 * kScanBig) {
    const int base = t0 + threadIdx.x * 4;
    int v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = (base + k < n) ? in[base + k] : 0;
      sum += v[k];
    }
    int x = sum;
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wid] = x;
    __syncthreads();
    int wbase = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kScanBig / 64; ++w) {
      if (w < wid) wbase += wsum[w];
      tot += wsum[w];
    }
    __syncthreads();   // wsum is rewritten by the next tile
    int ex = carry + wbase + x - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (base + k < n) out[base + k] = ex;
      ex += v[k];
    }
    carry += tot;
  }
}

size_t scan_temp_ints(int n) {
  const size_t tiles = (size_t)(n + kScanTile - 1) / kScanTile;
  if (tiles <= 1) return 1;
  return 2 * tiles + scan_temp_ints((int)tiles);
}

void launch_exclusive_scan(const int* in, int* out, int n, int* tmp, hipStream_t s) {
  if (n <= 0) return;
  const int tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles > 1 && n <= kScanSingleMax) {
    const ScanArgs a = {{in, nullptr}, {out, nullptr}, n};
    hipLaunchKernelGGL(k_scan_single, dim3(1), dim3(kScanBig), 0, s, a);
    return;
  }
  hipLaunchKernelGGL(k_scan_tiles, dim3(tiles), dim3(kBlock), 0, s, in, out, n, tmp);
  if (tiles == 1) return;
  launch_exclusive_scan(tmp, tmp + tiles, tiles, tmp + 2 * tiles, s);
  hipLaunchKernelGGL(k_scan_add, dim3(tiles), dim3(kBlock), 0, s, out, n,
                     (const int*)(tmp + tiles));
}

void launch_exclusive_scan2(const int* in0, int* out0, const int* in1, int* out1, int n, int* tmp,
                            hipStream_t s) {
  if (n <= 0) return;
  if (n <= kScanSingleMax) {
    const ScanArgs a = {{in0, in1}, {out0, out1}, n};
    hipLaunchKernelGGL(k_scan_single, dim3(2), dim3(kScanBig), 0, s, a);
    return;
  }
  launch_exclusive_scan(in0, out0, n, tmp, s);
  launch_exclusive_scan(in1, out1, n, tmp, s);
}

// ------------------------------------------------------------ binning
// Coordinate wrapped into [0, L).  Coordinates beyond kMaxBoxes box edges
// (rejected by the binning: the wrap has lost its precision there) map to
// 0, so that work queued before the error is read back indexes in bounds.
constexpr double kMaxBoxes = 1e6;
__device__ __forceinline__ double wrap(double x, double L, double iL) {
  double w = x - L * floor(x * iL);
  w = (w >= L) ? w - L : w;
  return (w > -L && w < L) ? w : 0.0;
}

// Polarizable: a nonzero tensor.
__device__ __forceinline__ bool nonzero6(const double* al) {
  bool pol = false;
#pragma unroll
  for (int k = 0; k < 6; ++k) pol = pol || al[k] != 0.0;
  return pol;
}

// Neighbouring caller indices are usually neighbouring sites (a molecule's
// sites, molecules laid out in space order), so the counters are
// incremented per wavefront run of equal keys.  A site's slot in its cell is
// the old value of the cell's counter (in no particular order: the cells are
// sorted afterwards); a second counter takes the cell's polarizable sites.
// Molecules are counted once per set of ids (mol_count given).
__global__ void k_bin(BinArgs a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const bool act = c < a.n;
  int cell = 0, m = -1;
  if (act) {
    const double x0 = a.xyz[3 * c], x1 = a.xyz[3 * c + 1], x2 = a.xyz[3 * c + 2];
    if (!isfinite(x0) || !isfinite(x1) || !isfinite(x2)) atomicOr(a.err, 8);
    if (a.periodic && !(fabs(x0) <= kMaxBoxes * a.box[0] && fabs(x1) <= kMaxBoxes * a.box[1] &&
                        fabs(x2) <= kMaxBoxes * a.box[2]))
      atomicOr(a.err, 8);
    if (a.periodic) {
      int ci[3];
      for (int d = 0; d < 3; ++d) {
        double w = wrap(a.xyz[3 * c + d], a.box[d], a.ibox[d]);
        int k = (int)(w * a.nc[d] * a.ibox[d]);
        ci[d] = k >= a.nc[d] ? a.nc[d] - 1 : (k < 0 ? 0 : k);
      }
      cell = ci[0] + a.nc[0] * (ci[1] + a.nc[1] * ci[2]);
    }
    m = a.mol[c];
    if (!(m >= 0 && m < a.n)) atomicOr(a.err, 2);
  }
  if (a.periodic) {
    const int slot = wave_atomic_inc(a.cell_count, cell, act);
    if (act) a.cell_slot[c] = make_int2(cell, slot);
    wave_atomic_inc(a.pol_count, cell, act && nonzero6(a.alpha + 6 * (size_t)c));
  }
  if (a.mol_count) wave_atomic_inc(a.mol_count, m, act && m >= 0 && m < a.n);
}

__global__ void k_scatter(const int2* cell_slot, const int* cell_start, int* perm, int n) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const int2 q = cell_slot[c];
  perm[cell_start[q.x] + q.y] = c;
}

// Sorts the n entries at seg (distinct indices) in increasing order by one
// wavefront, which makes the order independent of the order in which the
// binning's atomics ran: the entries are ranked in LDS (rank = number of
// smaller entries); segments too large for the LDS buffer fall back to an
// insertion sort by one lane.
constexpr int kSortLds = 256;
__device__ __forceinline__ void sort_segment(int* seg, int n, int* v) {
  if (n <= kSortLds) {
    for (int k = threadIdx.x; k < n; k += 64) v[k] = seg[k];
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += 64) {
      const int x = v[k];
      int r = 0;
      for (int m = 0; m < n; ++m) r += v[m] < x ? 1 : 0;
      seg[r] = x;
    }
  } else if (threadIdx.x == 0) {
    for (int i = 1; i < n; ++i) {
      const int x = seg[i];
      int j = i - 1;
      while (j >= 0 && seg[j] > x) {
        seg[j + 1] = seg[j];
        --j;
      }
      seg[j + 1] = x;
    }
  }
}

// Segments of two lists, one wavefront each: blocks [0, nseg) those of the
// first, [nseg, 2 nseg) those of the second.
__global__ __launch_bounds__(64) void k_sort_segments(const int* start0, int* v0,
                                                      const int* start1, int* v1, int nseg) {
  __shared__ int v[kSortLds];
  const bool second = (int)blockIdx.x >= nseg;
  const int b = blockIdx.x - (second ? nseg : 0);
  const int* start = second ? start1 : start0;
  int* perm = second ? v1 : v0;
  sort_segment(perm + start[b], start[b + 1] - start[b], v);
}

// Clusters: one cell in caller order, what the counting sort would give
// (its one-cell segment is past the rank sort's LDS buffer from 257 sites
// on: 5.9 ms for 400 sites, against 3 us here).
__global__ void k_one_cell(int* perm, int* cell_start, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) perm[i] = i;
  if (i == 0) { cell_start[0] = 0; cell_start[1] = n; }
}

void launch_one_cell(int* perm, int* cell_start, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_one_cell, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, perm,
                     cell_start, n);
}

__global__ void k_sum_ints(const int* v, int n, unsigned long long* out) {
  unsigned long long m = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    m += (unsigned long long)v[i];
  for (int off = 32; off > 0; off >>= 1) m += __shfl_xor(m, off, 64);
  if ((threadIdx.x & 63) == 0) atomicAdd(out, m);
}

void launch_sum_ints(const int* v, int n, unsigned long long* out, hipStream_t s) {
  int blocks = (n + kBlock - 1) / kBlock;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_sum_ints, dim3(blocks), dim3(kBlock), 0, s, v, n, out);
}

void launch_bin(const BinArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_bin, dim3((a.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
}
void launch_scatter(const int2* cell_slot, const int* cell_start, int* perm, int n,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_scatter, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, cell_slot,
                     cell_start, perm, n);
}
void launch_sort_segments(const int* start0, int* v0, const int* start1, int* v1, int nseg,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_sort_segments, dim3(2 * nseg), dim3(64), 0, s, start0, v0, start1, v1, nseg);
}
// ------------------------------------------------------------ records
// Positions (wrapped when periodic) and molecule ids in sorted order; the
// inverse permutation.  A non-finite coordinate (flagged by the binning, the
// call then fails) is stored as 0 and an out-of-range molecule id as 0, so
// that every kernel queued before the error is read back indexes in bounds.
__device__ __forceinline__ void rec_pos_of(const RecArgs& a, int i, int c, double xyz[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double v = a.xyz[3 * c + k];
    if (!isfinite(v)) v = 0.0;
    if (a.periodic) v = wrap(v, a.box[k], a.ibox[k]);
    xyz[k] = v;
  }
  const int m = a.mol[c];
  a.mol_s[i] = (m >= 0 && m < a.n) ? m : 0;
  a.inv_perm[c] = i;
}
// Multipoles of caller site c: q, d, Theta (zero where not given).
__device__ __forceinline__ void rec_mult_of(const RecArgs& a, int c, double& q, double d[3],
                                            double t[6]) {
  q = a.q ? a.q[c] : 0.0;
  for (int k = 0; k < 3; ++k) d[k] = a.dip ? a.dip[3 * c + k] : 0.0;
  for (int k = 0; k < 6; ++k) t[k] = a.quad ? a.quad[6 * c + k] : 0.0;
}
__device__ __forceinline__ void rec_mult_store(const RecArgs& a, int i, const double d[3],
                                               const double t[6]) {
  a.sth[i] = make_double4(t[0], t[1], t[2], t[3]);
  a.sth2[i] = make_double2(t[4], t[5]);
  a.sth32[i] = make_float4((float)t[0], (float)t[1], (float)t[2], (float)t[3]);
  a.sth232[i] = make_float2((float)t[4], (float)t[5]);
}
// Polarizability of caller site c: s = abar^-1/2 (0 when not polarizable);
// writes the Thole factor and the polarizable flag of sorted site i.
__device__ __forceinline__ double rec_pol_of(const RecArgs& a, int i, int c) {
  const double* al = a.alpha + 6 * (size_t)c;
  const bool pol = nonzero6(al);
  const double abar = (al[0] + al[3] + al[5]) / 3.0;
  a.sa[i] = a.thole ? a.thole[c] : a.thole_default;
  a.is_pol[i] = pol ? 1 : 0;
  return pol && abar > 0.0 ? 1.0 / sqrt(abar) : 0.0;
}

__global__ void k_rec_mult(RecArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  double q, d[3], t[6];
  rec_mult_of(a, a.perm[i], q, d, t);
  double4 p = a.sp[i];
  p.w = q;
  a.sp[i] = p;
  float4 p32 = a.sp32[i];
  p32.w = (float)q;
  a.sp32[i] = p32;
  double4 dd = a.sd[i];
  dd.x = d[0]; dd.y = d[1]; dd.z = d[2];
  a.sd[i] = dd;
  float4 dd32 = a.sd32[i];
  dd32.x = (float)d[0]; dd32.y = (float)d[1]; dd32.z = (float)d[2];
  a.sd32[i] = dd32;
  rec_mult_store(a, i, d, t);
}

// Polarizability records: s = abar^-1/2 (0 when not polarizable), Thole
// factor, polarizable flag.
__global__ void k_rec_pol(RecArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const double s = rec_pol_of(a, i, a.perm[i]);
  double4 dd = a.sd[i];
  dd.w = s;
  a.sd[i] = dd;
  float4 dd32 = a.sd32[i];
  dd32.w = (float)s;
  a.sd32[i] = dd32;
}

// After a re-sort all three records change: written whole.
__device__ __forceinline__ void rec_all_of(const RecArgs& a, int i, int c) {
  double x[3], q, d[3], t[6];
  rec_pos_of(a, i, c, x);
  rec_mult_of(a, c, q, d, t);
  const double s = rec_pol_of(a, i, c);
  a.sp[i] = make_double4(x[0], x[1], x[2], q);
  a.sp32[i] = make_float4((float)x[0], (float)x[1], (float)x[2], (float)q);
  a.sd[i] = make_double4(d[0], d[1], d[2], s);
  a.sd32[i] = make_float4((float)d[0], (float)d[1], (float)d[2], (float)s);
  rec_mult_store(a, i, d, t);
}

__global__ void k_rec_all(RecArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.n) rec_all_of(a, i, a.perm[i]);
}

// Polarizable records of sorted site i (caller site c) at polarizable index
// pi, including alpha^-1 (checked symmetric positive definite).
__device__ __forceinline__ void rec_polsite_of(const RecArgs& a, int i, int c, int pi) {
  a.polsite[pi] = i;
  const double4 p = a.sp[i];
  const double s = a.sd[i].w;
  a.pp[pi] = make_double4(p.x, p.y, p.z, s);
  a.pp32[pi] = make_float4((float)p.x, (float)p.y, (float)p.z, (float)s);
  a.pa[pi] = a.sa[i];
  const double* al = a.alpha + 6 * c;
  const double xx = al[0], xy = al[1], xz = al[2], yy = al[3], yz = al[4], zz = al[5];
#pragma unroll
  for (int k = 0; k < 6; ++k) a.alpha_s[6 * pi + k] = al[k];
  // Cholesky-type positivity test: leading principal minors > 0
  const double m1 = xx, m2 = xx * yy - xy * xy;
  const double det = xx * (yy * zz - yz * yz) - xy * (xy * zz - yz * xz) + xz * (xy * yz - yy * xz);
  if (!(m1 > 0.0 && m2 > 0.0 && det > 0.0)) atomicOr(a.err, 4);
  const double id = 1.0 / det;
  a.ainv_s[6 * pi + 0] = (yy * zz - yz * yz) * id;
  a.ainv_s[6 * pi + 1] = (xz * yz - xy * zz) * id;
  a.ainv_s[6 * pi + 2] = (xy * yz - xz * yy) * id;
  a.ainv_s[6 * pi + 3] = (xx * zz - xz * xz) * id;
  a.ainv_s[6 * pi + 4] = (xy * xz - xx * yz) * id;
  a.ainv_s[6 * pi + 5] = (xx * yy - xy * xy) * id;
}

// After the scan of is_pol: polarizable index maps and records.
__global__ void k_rec_polsites(RecArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const bool pol = a.is_pol[i] != 0;
  const int pi = a.pol_scan[i];
  a.polidx[i] = pol ? pi : -1;
  if (pol) rec_polsite_of(a, i, a.perm[i], pi);
}

// A cell's sites (periodic re-sort), one wavefront per cell: sorted by caller
// index, then every record and polarizable index in one pass.  Sort, records,
// a scan over all sites and the polarizable records were four to six
// launches, each little more than its launch time below 32,000 waters; with
// the two brick lists binned together (15 launches fewer in all) a step of
// 216 waters went from 1211 to 1166 us, of 32,000 from 4933 to 4903 us.
__global__ __launch_bounds__(64) void k_cell_records(RecArgs a, const int* cell_start,
                                                     const int* pol_start, int* perm) {
  __shared__ int v[kSortLds];
  const int cell = blockIdx.x, lane = threadIdx.x;
  const int s = cell_start[cell], n = cell_start[cell + 1] - s;
  sort_segment(perm + s, n, v);
  __syncthreads();
  int run = pol_start[cell];
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int i = s + k0 + lane;
    const bool on = k0 + lane < n;
    const int c = on ? perm[i] : 0;
    const bool pol = on && nonzero6(a.alpha + 6 * (size_t)c);
    const unsigned long long m = __ballot(pol);
    if (on) {
      rec_all_of(a, i, c);
      const int pi = lanes_below(m, run);
      a.polidx[i] = pol ? pi : -1;
      if (pol) rec_polsite_of(a, i, c, pi);
    }
    run += __popcll(m);
  }
}

void launch_cell_records(const RecArgs& a, const int* cell_start, const int* pol_start, int ncell,
                         int* perm, hipStream_t s) {
  hipLaunchKernelGGL(k_cell_records, dim3(ncell), dim3(64), 0, s, a, cell_start, pol_start, perm);
}
void launch_rec_all(const RecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_all, dim3((a.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
}
void launch_rec_mult(const RecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_mult, dim3((a.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
}
void launch_rec_pol(const RecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_pol, dim3((a.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
}
void launch_rec_polsites(const RecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_polsites, dim3((a.n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
}

// Extremes over the polarizable sites: block maxima / minima combined with
// atomics on the IEEE bit patterns (order-preserving for non-negative
// doubles), so the result does not depend on block order.  out must hold
// 0 and +inf beforehand.
__global__ __launch_bounds__(kBlock) void k_pol_extents(RecArgs a, unsigned long long* out) {
  __shared__ double smax[kBlock], smin[kBlock];
  double amax = 0.0, tmin = INFINITY;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < a.n; i += gridDim.x * kBlock) {
    if (!a.is_pol[i]) continue;
    const double s = a.sd[i].w;   // 1 / sqrt(mean polarizability)
    amax = fmax(amax, 1.0 / (s * s));
    tmin = fmin(tmin, fmax(a.sa[i], 0.0));
  }
  smax[threadIdx.x] = amax;
  smin[threadIdx.x] = tmin;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + w]);
      smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomicMax(&out[0], (unsigned long long)__double_as_longlong(smax[0]));
    atomicMin(&out[1], (unsigned long long)__double_as_longlong(smin[0]));
  }
}

void launch_pol_extents(const RecArgs& a, double* out, hipStream_t s) {
  unsigned long long* o = reinterpret_cast<unsigned long long*>(out);
  // 0.0 and +inf
  launch_fill_int(reinterpret_cast<int*>(o), 0, 3, s);
  launch_fill_int(reinterpret_cast<int*>(o) + 3, 0x7ff00000, 1, s);
  int blocks = (a.n + kBlock - 1) / kBlock;
  blocks = blocks < 1 ? 1 : (blocks > 256 ? 256 : blocks);
  hipLaunchKernelGGL(k_pol_extents, dim3(blocks), dim3(kBlock), 0, s, a, o);
}

// ------------------------------------------------------------ neighbour lists
// One wavefront builds the rows of one slice of a cell's sites: the cell's
// sites are dealt to `slices` wavefronts in contiguous runs (launch_nlist's
// caller picks the count, nlist_slices), and lists and their order do not
// depend on it.  Bound by instruction issue where the wavefronts fill the
// SIMDs (0.6 of the vector issue peak at 32,000 waters: 486 us, against 645
// with a branch per chunk and the chunks loaded in turn) and by the length of one
// wavefront's chain of candidate chunks where they do not: with one
// wavefront per cell the build took 300 us at 4,096 waters, 770 us at 1,001
// and 1.3 ms for a cluster of 80 (one cell), and whole evaluations went
// 1.98 -> 1.81, 2.70 -> 2.02 and (with k_one_cell) 4.59 -> 0.47 ms.
//  * the 5 x 5 rows of the stencil give at most 50 runs of consecutive
//    cells, each with a fixed periodic image shift (the stencil reaches a
//    wrapped cell through exactly one image), so a candidate's displacement
//    is x_i - (x_j + shift) without a per-pair rint.  Along an axis of fewer
//    than five cells every cell is a candidate once and the displacement is
//    brought to the nearest image per pair instead (NI); a cluster is one
//    cell without images;
//  * the runs are concatenated into one virtual candidate range, taken
//    kNlG chunks of 64 at a time into registers (a lane finds its run by
//    binary search over the run offsets), so chunks are full;
//  * each i-site's five running counts live in lane t and are read once per
//    pass over those chunks into wave-uniform (scalar) registers, so a
//    candidate chunk costs the distance test, the lane masks and the slot
//    arithmetic of its hits, about 36 instructions without a branch (the few
//    passes that hold the site's own molecule take one); hits are compacted
//    in lane order;
//  * the slice's count maxima go to its own slot of cellmax (plain stores;
//    launch_cellmax_reduce folds them), not to one atomic per wavefront on
//    four shared addresses.
constexpr int kNlIB = 64;   // i-sites handled per pass (one per lane)
constexpr int kNlG = 4;     // candidate chunks per pass over the i-sites

__device__ __forceinline__ int rl(int v, int t) { return __builtin_amdgcn_readlane(v, t); }
// lane masks straight from one vector compare (predicate codes of the
// compiler's compare intrinsics: ordered less-than; signed equal, >=)
constexpr int kCmpOLT = 4, kCmpEQ = 32, kCmpSGE = 39;
__device__ __forceinline__ unsigned long long mask_lt(double a, double b) {
  return __builtin_amdgcn_fcmp(a, b, kCmpOLT);
}
__device__ __forceinline__ unsigned long long mask_eq(int a, int b) {
  return __builtin_amdgcn_sicmp(a, b, kCmpEQ);
}

template <bool NI>
__global__ __launch_bounds__(64) void k_nlist(NlistArgs a) {
  __shared__ double xi[kNlIB], yi[kNlIB], zi[kNlIB];
  __shared__ int run_s[50], run_off[64], run_code[50];
  const int lane = threadIdx.x;
  const int cell = blockIdx.x / a.slices, slice = blockIdx.x - cell * a.slices;
  const int nc0 = a.nc[0], nc1 = a.nc[1], nc2 = a.nc[2];
  const int cx = cell % nc0, cy = (cell / nc0) % nc1, cz = cell / (nc0 * nc1);
  const int c0 = a.cell_start[cell], c1 = a.cell_start[cell + 1];
  const int per = (c1 - c0 + a.slices - 1) / a.slices;
  const int i0 = min(c1, c0 + slice * per), i1 = min(c1, i0 + per);
  if (i0 >= i1) {
    if (lane == 0) a.cellmax[blockIdx.x] = make_int4(0, 0, 0, 0);
    return;
  }
  const double L0 = a.box[0], L1 = a.box[1], L2 = a.box[2];
  // axes taken whole, and the box edges their displacements wrap by (0: no
  // wrap along this axis)
  const bool w0 = nc0 < 5, w1 = nc1 < 5, w2 = nc2 < 5;
  const double W0 = NI && w0 ? L0 : 0.0, W1 = NI && w1 ? L1 : 0.0, W2 = NI && w2 ? L2 : 0.0;
  const double iW0 = NI && w0 ? a.ibox[0] : 0.0, iW1 = NI && w1 ? a.ibox[1] : 0.0,
               iW2 = NI && w2 ? a.ibox[2] : 0.0;
  const int sy = w1 ? nc1 : 5, sz = w2 ? nc2 : 5;
  int len0 = 0, len1 = 0;   // lengths of this lane's two runs
  if (lane < sy * sz) {
    int zz, yy, zc = 1, yc = 1;   // image codes: 0 below, 1 home, 2 above
    if (w2) zz = lane / sy;
    else {
      zz = cz + lane / sy - 2;
      if (zz < 0) { zz += nc2; zc = 0; } else if (zz >= nc2) { zz -= nc2; zc = 2; }
    }
    if (w1) yy = lane % sy;
    else {
      yy = cy + lane % sy - 2;
      if (yy < 0) { yy += nc1; yc = 0; } else if (yy >= nc1) { yy -= nc1; yc = 2; }
    }
    const int row = nc0 * (yy + nc1 * zz);
    const int x0 = cx - 2, x1 = cx + 2;
    int f0, l0, k0, f1 = 0, l1 = -1, k1 = 1;   // cell ranges [f, l] and x image codes
    if (w0) { f0 = 0; l0 = nc0 - 1; k0 = 1; }
    else if (x0 >= 0 && x1 < nc0) { f0 = x0; l0 = x1; k0 = 1; }
    else if (x0 < 0) { f0 = 0; l0 = x1; k0 = 1; f1 = nc0 + x0; l1 = nc0 - 1; k1 = 0; }
    else { f0 = x0; l0 = nc0 - 1; k0 = 1; f1 = 0; l1 = x1 - nc0; k1 = 2; }
    const int yzc = 4 * yc + 16 * zc;
    run_s[2 * lane] = a.cell_start[row + f0];
    len0 = a.cell_start[row + l0 + 1] - a.cell_start[row + f0];
    run_code[2 * lane] = k0 + yzc;
    if (l1 >= f1) {
      run_s[2 * lane + 1] = a.cell_start[row + f1];
      len1 = a.cell_start[row + l1 + 1] - a.cell_start[row + f1];
    } else {
      run_s[2 * lane + 1] = 0;
    }
    run_code[2 * lane + 1] = k1 + yzc;
  }
  {
    int x = len0 + len1;   // inclusive scan over the rows
    for (int off = 1; off < 32; off <<= 1) {
      const int y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane < 25) {
      run_off[2 * lane + 1] = x - len1;
      run_off[2 * lane + 2] = x;
    }
    if (lane == 0) run_off[0] = 0;
    if (lane > 50) run_off[lane] = INT_MAX;
  }
  __syncthreads();
  const int ncand = run_off[50];
  const unsigned cap_all = a.cap_all;
  const int cap_in = a.cap_in, cap_pol = a.cap_pol, cap_ipol = a.cap_ipol;
  const double cut2 = a.cutoff2, split2 = a.rsplit2;
  int4 mx = make_int4(0, 0, 0, 0);   // the slice's count maxima
  for (int ib = i0; ib < i1; ib += kNlIB) {
    const int ni = min(kNlIB, i1 - ib);
    // i-site `lane`: position in LDS (read back as a broadcast), molecule
    // and polarizable index in registers
    int mol_v = -1, pol_v = -1;
    if (lane < ni) {
      const double4 p = a.sp[ib + lane];
      xi[lane] = p.x; yi[lane] = p.y; zi[lane] = p.z;
      mol_v = a.mol_s[ib + lane];
      pol_v = a.polidx[ib + lane];
    }
    __syncthreads();
    // index of the pass's first polarizable site
    const unsigned long long pols = __builtin_amdgcn_sicmp(pol_v, 0, kCmpSGE);
    const int pol0 = pols ? rl(pol_v, __builtin_ctzll(pols)) : 0;
    // counts of i-site `lane`: all near (cnt0) and far (cntf), in, pol, ipol
    int cnt0 = 0, cntf = 0, cnt1 = 0, cnt2 = 0, cnt3 = 0;
    for (int c = 0; c < ncand; c += 64 * kNlG) {
      // a lane past the candidates sits at infinity in no molecule: it
      // never tests as a neighbour (also of a cluster's infinite cutoff)
      double xj[kNlG], yj[kNlG], zj[kNlG];
      int jj[kNlG], molj[kNlG], polj[kNlG];
      unsigned long long pjm[kNlG];
      // the chunks' searches (last run that starts at or before the
      // candidate) and loads side by side, without branches: one after the
      // other they were a third of a wavefront's time
      int run[kNlG];
      double4 pj[kNlG];
#pragma unroll
      for (int g = 0; g < kNlG; ++g) run[g] = 0;
#pragma unroll
      for (int step = 32; step; step >>= 1)
#pragma unroll
        for (int g = 0; g < kNlG; ++g)
          if (run_off[run[g] + step] <= c + g * 64 + lane) run[g] += step;
#pragma unroll
      for (int g = 0; g < kNlG; ++g) {
        const int cidx = c + g * 64 + lane;
        run[g] = cidx < ncand ? run[g] : 0;
        jj[g] = cidx < ncand ? run_s[run[g]] + (cidx - run_off[run[g]]) : 0;
        pj[g] = a.sp[jj[g]];
        molj[g] = a.mol_s[jj[g]];
        polj[g] = a.polidx[jj[g]];
      }
#pragma unroll
      for (int g = 0; g < kNlG; ++g) {
        const bool on = c + g * 64 + lane < ncand;
        const int code = run_code[run[g]];
        xj[g] = on ? pj[g].x + L0 * (double)((code & 3) - 1) : (double)INFINITY;
        yj[g] = on ? pj[g].y + L1 * (double)(((code >> 2) & 3) - 1) : (double)INFINITY;
        zj[g] = on ? pj[g].z + L2 * (double)((code >> 4) - 1) : (double)INFINITY;
        jj[g] = on ? jj[g] : -1;
        molj[g] = on ? molj[g] : -1;
        polj[g] = on ? polj[g] : -1;
        pjm[g] = __builtin_amdgcn_sicmp(polj[g], 0, kCmpSGE);
      }
      // rows of the sites in turn: consecutive, as polarizable indices are
      int* row_all = a.nb_all + (size_t)ib * cap_all;
      int* row_pol = a.nb_pol + (size_t)pol0 * cap_pol;
      for (int t = 0; t < ni; ++t) {
        const double x = xi[t], y = yi[t], z = zi[t];
        const int mi = rl(mol_v, t);
        // lane masks of every chunk before any of them is used, straight
        // line: cut (intermolecular within the cutoff), near of them, mol
        unsigned long long cut[kNlG], near[kNlG], mol[kNlG], any = 0ull;
#pragma unroll
        for (int g = 0; g < kNlG; ++g) {
          double dx = x - xj[g], dy = y - yj[g], dz = z - zj[g];
          if (NI) {
            dx -= W0 * rint(dx * iW0);
            dy -= W1 * rint(dy * iW1);
            dz -= W2 * rint(dz * iW2);
          }
          const double r2 = dx * dx + dy * dy + dz * dz;
          mol[g] = mask_eq(molj[g], mi);
          cut[g] = mask_lt(r2, cut2) & ~mol[g];
          near[g] = mask_lt(r2, split2) & cut[g];
          any |= mol[g];
        }
        const bool pol = rl(pol_v, t) >= 0;
        // site t's counts, wave-uniform for the chunks of this pass; a
        // lane's slot is the count plus the lower lanes of its mask; near
        // entries from the front of the row, far ones from its back
        int k0 = rl(cnt0, t), kf = rl(cntf, t);
#pragma unroll
        for (int g = 0; g < kNlG; ++g) {
          const unsigned long long far = cut[g] & ~near[g];
          const int kn = lanes_below(near[g], k0), kb = lanes_below(far, kf);
          const unsigned k = __builtin_amdgcn_inverse_ballot_w64(near[g])
                                 ? (unsigned)kn : cap_all - 1u - (unsigned)kb;
          if (__builtin_amdgcn_inverse_ballot_w64(cut[g]) && k < cap_all) row_all[k] = jj[g];
          k0 += __popcll(near[g]);
          kf += __popcll(far);
        }
        const bool me = lane == t;
        cnt0 = me ? k0 : cnt0;
        cntf = me ? kf : cntf;
        if (pol) {
          int k2 = rl(cnt2, t);
#pragma unroll
          for (int g = 0; g < kNlG; ++g) {
            const unsigned long long m = cut[g] & pjm[g];
            const int k = lanes_below(m, k2);
            if (__builtin_amdgcn_inverse_ballot_w64(m) && k < cap_pol) row_pol[(unsigned)k] = polj[g];
            k2 += __popcll(m);
          }
          cnt2 = me ? k2 : cnt2;
        }
        if (any) {   // same molecule, not site t itself
          const int i = ib + t;
          int k1 = rl(cnt1, t), k3 = rl(cnt3, t);
          int* row_in = a.nb_in + (size_t)i * cap_in;
          int* row_ipol = a.nb_ipol + (size_t)(pol ? rl(pol_v, t) : 0) * cap_ipol;
#pragma unroll
          for (int g = 0; g < kNlG; ++g) {
            const unsigned long long b1 = mol[g] & ~mask_eq(jj[g], i);
            const unsigned long long b3 = pol ? b1 & pjm[g] : 0ull;
            const int k = lanes_below(b1, k1), kp = lanes_below(b3, k3);
            if (__builtin_amdgcn_inverse_ballot_w64(b1) && k < cap_in) row_in[(unsigned)k] = jj[g];
            if (__builtin_amdgcn_inverse_ballot_w64(b3) && kp < cap_ipol)
              row_ipol[(unsigned)kp] = polj[g];
            k1 += __popcll(b1);
            k3 += __popcll(b3);
          }
          cnt1 = me ? k1 : cnt1;
          cnt3 = me ? k3 : cnt3;
        }
        row_all += cap_all;
        if (pol) row_pol += cap_pol;
      }
    }
    if (lane < ni) {
      const int i = ib + lane;
      a.nc_all[i] = cnt0 + cntf;
      a.nc_near[i] = cnt0;
      a.nc_in[i] = cnt1;
      if (pol_v >= 0) {
        a.nc_pol[pol_v] = cnt2;
        a.nc_ipol[pol_v] = cnt3;
      }
      if (cnt1 != a.mol_count[mol_v] - 1) atomicOr(a.err, 1);
    }
    mx.x = max(mx.x, wave_max(lane < ni ? cnt0 + cntf : 0));
    mx.y = max(mx.y, wave_max(lane < ni ? cnt1 : 0));
    mx.z = max(mx.z, wave_max(pol_v >= 0 ? cnt2 : 0));
    mx.w = max(mx.w, wave_max(pol_v >= 0 ? cnt3 : 0));
    __syncthreads();
  }
  if (lane == 0) a.cellmax[blockIdx.x] = mx;
}

__global__ __launch_bounds__(1024) void k_cellmax_reduce(const int4* cellmax, int count, int* out) {
  __shared__ int4 part[16];
  int4 m = make_int4(0, 0, 0, 0);
  for (int k = threadIdx.x; k < count; k += blockDim.x) {
    const int4 v = cellmax[k];
    m.x = max(m.x, v.x); m.y = max(m.y, v.y); m.z = max(m.z, v.z); m.w = max(m.w, v.w);
  }
  m.x = wave_max(m.x); m.y = wave_max(m.y); m.z = wave_max(m.z); m.w = wave_max(m.w);
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 0) part[w] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    int4 r = part[0];
    for (int k = 1; k < nw; ++k) {
      r.x = max(r.x, part[k].x); r.y = max(r.y, part[k].y);
      r.z = max(r.z, part[k].z); r.w = max(r.w, part[k].w);
    }
    out[0] = r.x; out[1] = r.y; out[2] = r.z; out[3] = r.w;
  }
}

void launch_cellmax_reduce(const int4* cellmax, int count, int* out, hipStream_t s) {
  hipLaunchKernelGGL(k_cellmax_reduce, dim3(1), dim3(1024), 0, s, cellmax, count, out);
}

// Wavefronts per cell: enough for kNlWaves in all, at most one per site of
// an average cell; two up to twice kNlWaves cells, where one each are too few
// rounds of the 5,120 that fit to even out (9,261 cells: 546 against 486 us;
// three take 520, as every slice loads the cell's candidates).  One / two: 5,832
// cells 335 / 307 us, 8,000 422 / 392, 13,824 617 / 591; at 17,576, past the line,
// 747 / 711 in one run and 706 / 717 in another.
int nlist_slices(int n, int ncell) {
  const int per_cell = (n + ncell - 1) / ncell;
  return std::max(1, std::min(per_cell, std::max(kNlWaves / ncell, ncell < 2 * kNlWaves ? 2 : 1)));
}

void launch_nlist(const NlistArgs& a, int ncell, hipStream_t s) {
  const dim3 g((unsigned)ncell * a.slices), b(64);
  // a cluster needs no images; one that is periodic along a short axis does
  if (a.periodic && (a.nc[0] < 5 || a.nc[1] < 5 || a.nc[2] < 5))
    hipLaunchKernelGGL(k_nlist<true>, g, b, 0, s, a);
  else
    hipLaunchKernelGGL(k_nlist<false>, g, b, 0, s, a);
}

}  // namespace sibfa
