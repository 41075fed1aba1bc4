// Lagrangian-Eulerian coupling on gfx950: marker setup, tile binning, spread S (and the fused
// dipole spread S~ = div S(q n) of the finite-difference discretisation), interpolation S*.
//
// Spread is owner-computes: one workgroup owns one tile of grid nodes, loads the markers whose
// 6-node window meets the tile into LDS, and every thread sums the contributions to its own
// nodes in registers.  There are no atomics on grid data, so the result is deterministic, and
// every tile (zeros included) is written exactly once with coalesced stores.
//
// Kernel windows: node indices s, s+1, ..., s+5 per axis with s = floor((X - origin)/h) - 2;
// the 4-point kernels are non-zero on the middle four, the 6-point B-spline on all six.
#include "kernels.h"

namespace ibdl {
namespace {


__device__ __forceinline__ double phi_eval(int kernel, double r) {
  const double a = fabs(r);
  if (kernel == KID_PESKIN4) {
    if (a <= 1.0) return (3.0 - 2.0 * a + sqrt(1.0 + 4.0 * a - 4.0 * a * a)) * 0.125;
    if (a < 2.0) return (5.0 - 2.0 * a - sqrt(fmax(-7.0 + 12.0 * a - 4.0 * a * a, 0.0))) * 0.125;
    return 0.0;
  }
  if (kernel == KID_COS4) return a < 2.0 ? 0.25 * (1.0 + cospi(0.5 * a)) : 0.0;
  // quintic B-spline, 6 points
  if (a <= 1.0) return 11.0 / 20.0 - a * a / 2.0 + a * a * a * a / 4.0 - a * a * a * a * a / 12.0;
  if (a <= 2.0)
    return 17.0 / 40.0 + 5.0 * a / 8.0 - 7.0 * a * a / 4.0 + 5.0 * a * a * a / 4.0 - 3.0 * a * a * a * a / 8.0 +
           a * a * a * a * a / 24.0;
  if (a < 3.0)
    return 81.0 / 40.0 - 27.0 * a / 8.0 + 9.0 * a * a / 4.0 - 3.0 * a * a * a / 4.0 + a * a * a * a / 8.0 -
           a * a * a * a * a / 120.0;
  return 0.0;
}

// d phi / d r, the derivative of each piece in |r| times the sign of r
__device__ __forceinline__ double dphi_eval(int kernel, double r) {
  const double a = fabs(r), sg = r < 0.0 ? -1.0 : 1.0;
  double v = 0.0;
  if (kernel == KID_PESKIN4) {
    if (a <= 1.0) v = (-2.0 + (4.0 - 8.0 * a) / (2.0 * sqrt(1.0 + 4.0 * a - 4.0 * a * a))) * 0.125;
    else if (a < 2.0) v = (-2.0 - (12.0 - 8.0 * a) / (2.0 * sqrt(fmax(-7.0 + 12.0 * a - 4.0 * a * a, 1e-300)))) * 0.125;
    return sg * v;
  }
  if (kernel == KID_COS4) return a < 2.0 ? -0.125 * M_PI * sinpi(0.5 * r) : 0.0;
  if (a <= 1.0) v = -a + a * a * a - 5.0 * a * a * a * a / 12.0;
  else if (a <= 2.0) v = 5.0 / 8.0 - 7.0 * a / 2.0 + 15.0 * a * a / 4.0 - 3.0 * a * a * a / 2.0 + 5.0 * a * a * a * a / 24.0;
  else if (a < 3.0) v = -27.0 / 8.0 + 9.0 * a / 2.0 - 9.0 * a * a / 4.0 + a * a * a / 2.0 - a * a * a * a / 24.0;
  return sg * v;
}

// ------------------------------------------------------------------ marker setup and binning
// Tiles met by a marker's 6-node window along each axis: tile indices j0 .. j0 + cnt - 1 (mod ntile).
__device__ __forceinline__ void marker_tiles(const MarkerGeom& g, const int* s, int (&j0)[3], int (&cnt)[3]) {
  for (int d = 0; d < 3; ++d) {
    if (d < g.dim) {
      j0[d] = s[d] / g.tile[d];
      cnt[d] = (s[d] + 5) / g.tile[d] - j0[d] + 1;
      if (cnt[d] > g.ntile[d]) cnt[d] = g.ntile[d];
    } else {
      j0[d] = 0;
      cnt[d] = 1;
    }
  }
}

__device__ __forceinline__ int tile_id(const MarkerGeom& g, const int (&j0)[3], int a, int b, int c) {
  const int tz = (j0[2] + a) % g.ntile[2], ty = (j0[1] + b) % g.ntile[1], tx = (j0[0] + c) % g.ntile[0];
  return (tz * g.ntile[1] + ty) * g.ntile[0] + tx;
}

// Four lanes per marker: lane d < 3 places the marker along axis d and evaluates that axis's weights (a
// chain which one thread per marker ran three times over on a few waves: 31 us at 18,500 markers in 3-D,
// now 21); all four then count the tiles.
__global__ __launch_bounds__(256) void k_marker_setup(MarkerGeom g, int kernel, int64_t n_ib,
                                                      const double* __restrict__ X, int* __restrict__ s,
                                                      double* __restrict__ f, double* __restrict__ wt,
                                                      int* __restrict__ tile_count, const int* __restrict__ pid) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = e >> 2;
  const int d = (int)(e & 3);
  const bool live = i < n_ib;
  int sd = 0;
  if (live && d < 3) {
    double fr = 0.0;
    if (d < g.dim) {
      const double n = (double)g.n[d];
      double xi = (X[i * g.dim + d] - g.origin[d]) / g.h;
      xi = xi - n * floor(xi / n);                 // wrap into [0, n)
      if (!(xi >= 0.0 && xi < n)) xi = 0.0;        // non-finite input: keep indices in range
      int bi = (int)floor(xi);
      if (bi >= g.n[d]) bi = g.n[d] - 1;
      fr = xi - (double)bi;
      sd = (bi - 2 + 2 * g.n[d]) & (g.n[d] - 1);
    }
    s[i * 3 + d] = sd;
    f[i * 3 + d] = fr;
    // kernel weights W[t] = phi((s + t) - X/h) on the 6-node window and centred differences
    // G[t] = (W[t+1] - W[t-1]) / 2h (W = 0 outside the window), per axis; unit weight off-dimension
    double w[8];
    w[0] = w[7] = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) w[t + 1] = d < g.dim ? phi_eval(kernel, (double)(t - 2) - fr) : (t == 2 ? 1.0 : 0.0);
    double* row = wt + (i * 3 + d) * 12;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      row[t] = w[t + 1];
      row[6 + t] = d < g.dim ? (w[t + 2] - w[t]) * (0.5 / g.h) : 0.0;
    }
  }
  const int l0 = (int)(threadIdx.x & 60);
  const int si[3] = {__shfl(sd, l0), __shfl(sd, l0 + 1), __shfl(sd, l0 + 2)};
  if (!live) return;
  int j0[3], nt[3];
  marker_tiles(g, si, j0, nt);
  const int toff = pid ? pid[i] * g.ntile[0] * g.ntile[1] * g.ntile[2] : 0;   // tiles of problem pid[i]
  for (int q = d; q < nt[0] * nt[1] * nt[2]; q += 4)
    atomicAdd(&tile_count[toff + tile_id(g, j0, q / (nt[0] * nt[1]), q / nt[0] % nt[1], q % nt[0])], 1);
}

// eight lanes per marker, one tile each (an atomic's round trip per tile, not one after another: 23 us at
// 18,500 markers in 3-D, now 19)
__global__ __launch_bounds__(256) void k_fill(MarkerGeom g, int64_t n_ib, const int* __restrict__ s,
                                              const int* __restrict__ off, int* __restrict__ cur,
                                              int* __restrict__ list, const int* __restrict__ pid) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = e >> 3;
  if (i >= n_ib) return;
  const int si[3] = {s[i * 3], s[i * 3 + 1], s[i * 3 + 2]};
  int j0[3], nt[3];
  marker_tiles(g, si, j0, nt);
  const int toff = pid ? pid[i] * g.ntile[0] * g.ntile[1] * g.ntile[2] : 0;
  for (int q = (int)(e & 7); q < nt[0] * nt[1] * nt[2]; q += 8) {
    const int id = toff + tile_id(g, j0, q / (nt[0] * nt[1]), q / nt[0] % nt[1], q % nt[0]);
    const int pos = off[id] + atomicAdd(&cur[id], 1);
    list[pos] = (int)i;
  }
}

// Exclusive prefix of v over a workgroup of 1024 threads; tot: the workgroup's sum.  Sixteen waves, each
// by shuffles, and their sums through s_w[16]: two barriers, the first of which also ends the last use.
template <typename V> __device__ __forceinline__ V block_scan(V v, V* s_w, V& tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  V x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const V t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  __syncthreads();
  if (lane == 63) s_w[wave] = x;
  __syncthreads();
  V before = 0;
  tot = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const V t = s_w[w];
    before += w < wave ? t : 0;
    tot += t;
  }
  return before + x - v;
}

constexpr int kScanItems = 4;   // consecutive items per thread and trip of the one-block scans

// exclusive scan of cnt[0..n) into off[0..n]; one block of 1024 threads
__global__ __launch_bounds__(1024) void k_scan(const int* __restrict__ cnt, int* __restrict__ off, int n) {
  __shared__ int s_w[16];
  int carry = 0;
  for (int base = 0; base < n; base += 1024 * kScanItems) {
    const int i0 = base + (int)threadIdx.x * kScanItems;
    int v[kScanItems], sum = 0, tot;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) sum += v[k] = i0 + k < n ? cnt[i0 + k] : 0;
    int o = carry + block_scan(sum, s_w, tot);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (i0 + k < n) off[i0 + k] = o;
      o += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) off[n] = carry;
}

// The tile lists' offsets (exclusive scan of the candidate counts) and the tiles with at least one
// candidate, in increasing order, with their list ranges; foff[n]: their number; cur cleared for k_fill.
// One block of 1024 threads, both scans in one 64-bit sum (number of busy tiles above, candidates below):
// 4,096 tiles in 5 us, where a kernel for the flags, two scans with two barriers a doubling, the list and
// a clearing took 26.
__global__ __launch_bounds__(1024) void k_bin_scan(const int* __restrict__ cnt, int* __restrict__ off,
                                                   int* __restrict__ foff, int4* __restrict__ busy,
                                                   int* __restrict__ cur, int n) {
  __shared__ unsigned long long s_w[16];
  unsigned long long carry = 0;
  for (int base = 0; base < n; base += 1024 * kScanItems) {
    const int i0 = base + (int)threadIdx.x * kScanItems;
    int v[kScanItems];
    unsigned long long sum = 0, tot;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      v[k] = i0 + k < n ? cnt[i0 + k] : 0;
      sum += ((unsigned long long)(v[k] > 0) << 32) + (unsigned)v[k];
    }
    const unsigned long long o = carry + block_scan(sum, s_w, tot);
    int fo = (int)(o >> 32), co = (int)(o & 0xffffffffu);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (i0 + k < n) {
        off[i0 + k] = co;
        cur[i0 + k] = 0;
        if (v[k] > 0) busy[fo++] = make_int4(i0 + k, co, co + v[k], 0);
      }
      co += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) {
    off[n] = (int)(carry & 0xffffffffu);
    foff[n] = (int)(carry >> 32);
  }
}

// per-precision weight table: (W[t], G[t]) pairs, t < 6, padded with zeros at t = 6, 7
template <typename T>
__global__ void k_wtab(const double* __restrict__ wt, int64_t n_ib, cplx<T>* __restrict__ tab) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // (marker, axis, tap)
  if (e >= n_ib * 24) return;
  const int64_t r = e >> 3;
  const int t = (int)(e & 7);
  tab[e] = t < 6 ? mk<cplx<T>>((T)wt[r * 12 + t], (T)wt[r * 12 + 6 + t]) : mk<cplx<T>>((T)0, (T)0);
}

// busy tiles along x of each listed row as a bit mask of seg_row_words words: bit t & 63 of word t >> 6
// for tile (t, strip of the row), t < ntx; one thread per row and word (its mask returned, 0 past the last)
__device__ __forceinline__ unsigned long long row_segments(const MarkerGeom& g, const int* __restrict__ tile_off,
                                                           const int* __restrict__ rows, int64_t nact, int64_t e,
                                                           unsigned long long* __restrict__ seg) {
  const int nw = seg_row_words(g);
  if (e >= nact * nw) return 0;
  const int64_t r = e / nw;
  const int t0 = 64 * (int)(e - r * nw);
  const int w = rows ? rows[r] : (int)r, y = w % g.n[1], z = w / g.n[1];
  // z counts planes, or problems of a batch in 2-D (tile[2] = 1 there): tiles are numbered
  // problem-major, so the strip index runs on across a batch's problems
  const int64_t strip = y / g.tile[1] + (int64_t)g.ntile[1] * (z / g.tile[2]);
  const int nt = g.ntile[0] - t0 < 64 ? g.ntile[0] - t0 : 64;
  const int* off = tile_off + strip * g.ntile[0] + t0;
  unsigned long long m = 0;
  for (int t = 0; t < nt; ++t)
    if (off[t + 1] > off[t]) m |= 1ull << t;
  seg[e] = m;
  return m;
}
__global__ __launch_bounds__(256) void k_row_segments(MarkerGeom g, const int* __restrict__ tile_off,
                                                      const int* __restrict__ rows, int64_t nact,
                                                      unsigned long long* __restrict__ seg) {
  row_segments(g, tile_off, rows, nact, (int64_t)blockIdx.x * 256 + threadIdx.x, seg);
}
// The masks of every row, and the number of bits set in those of the active rows (lim) to *host, pinned:
// the workgroups add (1 above, their bits below) to *count, and the last one has the sum.
__global__ __launch_bounds__(256) void k_all_row_segments(MarkerGeom g, const int* __restrict__ tile_off, int64_t nrows,
                                                          const int2* __restrict__ lim, unsigned long long* __restrict__ seg,
                                                          unsigned long long* count, int* __restrict__ host) {
  __shared__ int red[4];
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const unsigned long long m = row_segments(g, tile_off, nullptr, nrows, e, seg);
  int c = 0;
  if (m) {
    const int64_t r = e / seg_row_words(g);
    const int y = (int)(r % g.n[1]);
    const int2 l = lim[r / g.n[1]];
    if (y >= l.x && y <= l.y) c = __popcll(m);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long mine = (1ull << 32) + (unsigned)(red[0] + red[1] + red[2] + red[3]);
    const unsigned long long sum = atomicAdd(count, mine) + mine;
    if ((unsigned)(sum >> 32) == gridDim.x) *host = (int)(sum & 0xffffffffu);
  }
}

// The busy tiles in decreasing order of their candidate count (ties by tile id): the spread's
// workgroups then start with the longest tiles and end with the shortest, which evens out the
// CUs' finishing times.  Rank sort; *nptr = number of busy tiles.  A workgroup ranks kOrder tiles: its
// threads count over the tiles' list side by side, each against all kOrder (one thread per tile, the list
// staged in LDS: 42 us at 784 tiles, a serial chain of 784 reads on four workgroups; now 7).
// groups: the tiles (in tile-id order, i.e. in slabs) are first cut into the 8 XCD-contiguous
// ranges of xcd_chunk, and each range is ordered on its own, so that a spread reading entry
// xcd_chunk(b, n) gives each XCD one slab of neighbouring tiles, longest first; their markers'
// data then stay in that XCD's L2.
__device__ __forceinline__ int xcd_range_lo(int x, int n) {   // first index of XCD range x of [0, n)
  const int q = n / 8, r = n % 8;
  return x * q + (x < r ? x : r);
}
constexpr int kOrder = 8;
__global__ __launch_bounds__(256) void k_busy_order(const int4* __restrict__ in, const int* __restrict__ nptr,
                                                    int4* __restrict__ out, int groups) {
  __shared__ int s_rk[4][kOrder];
  const int n = *nptr;
  const int i0 = (int)blockIdx.x * kOrder;
  if (i0 >= n) return;
  int c[kOrder], lo[kOrder], hi[kOrder], rk[kOrder];
#pragma unroll
  for (int e = 0; e < kOrder; ++e) {
    const int i = i0 + e < n ? i0 + e : n - 1;
    const int4 v = in[i];
    c[e] = v.z - v.y;
    lo[e] = 0;
    hi[e] = n;
    rk[e] = 0;
    if (groups) {
      const int q = n / 8, r = n % 8;
      const int x = i < r * (q + 1) ? i / (q + 1) : r + (q > 0 ? (i - r * (q + 1)) / q : 0);
      lo[e] = xcd_range_lo(x, n);
      hi[e] = xcd_range_lo(x + 1, n);
    }
  }
  for (int k = lo[0] + (int)threadIdx.x; k < hi[kOrder - 1]; k += 256) {
    const int4 u = in[k];
    const int ck = u.z - u.y;
#pragma unroll
    for (int e = 0; e < kOrder; ++e)
      rk[e] += (k >= lo[e] && k < hi[e]) && ((ck > c[e]) || (ck == c[e] && k < i0 + e));
  }
#pragma unroll
  for (int e = 0; e < kOrder; ++e) {
    for (int o = 32; o > 0; o >>= 1) rk[e] += __shfl_xor(rk[e], o);
    if ((threadIdx.x & 63) == 0) s_rk[threadIdx.x >> 6][e] = rk[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kOrder; ++e)
    if ((int)threadIdx.x == e && i0 + e < n)
      out[lo[e] + s_rk[0][e] + s_rk[1][e] + s_rk[2][e] + s_rk[3][e]] = in[i0 + e];
}

// Sort each tile's marker list ascending (rank sort; marker indices in a tile are unique).  The list goes
// through LDS 256 entries at a time, four a read: the ranks come from broadcasts, not from memory (4,096
// tiles, 784 of them busy: 26 us with one load from memory per compared entry, now 15).
__global__ __launch_bounds__(256) void k_sort_tiles(const int* __restrict__ off, const int* __restrict__ tmp,
                                                    int* __restrict__ list) {
  __shared__ int4 s_v[64];
  const int b = off[blockIdx.x], L = off[blockIdx.x + 1] - b;
  for (int a0 = 0; a0 < L; a0 += 256) {
    const int a = a0 + (int)threadIdx.x;
    const int v = a < L ? tmp[b + a] : 0;
    int r = 0;
    for (int k0 = 0; k0 < L; k0 += 256) {
      const int k = k0 + (int)threadIdx.x;
      __syncthreads();
      reinterpret_cast<int*>(s_v)[threadIdx.x] = k < L ? tmp[b + k] : 0x7fffffff;
      __syncthreads();
      const int kn = ((L - k0 < 256 ? L - k0 : 256) + 3) / 4;
      for (int q = 0; q < kn; ++q) {
        const int4 u = s_v[q];
        r += (u.x < v) + (u.y < v) + (u.z < v) + (u.w < v);
      }
    }
    if (a < L) list[b + r] = v;
  }
}

// ------------------------------------------------------------------ spread
// Owner-computes spread with the candidate list of a tile split over the 4 waves of a workgroup:
// wave w accumulates candidates w, w+4, w+8, ... of the (sorted) list in registers, and the four
// partial sums are added in wave order at the end, so the result is deterministic.  The loader
// thread of each candidate evaluates the kernel weights W and the centred-difference weights G
// at the tile's own node positions (zero outside the marker's window), so the accumulation loop
// is branch-free and reads a handful of packed LDS vectors per candidate.
constexpr int kT3X = 16, kT3Y = 4, kT3Z = 8;   // 3-D tile; lane (x, y) owns a z-column of 8
constexpr int kT2X = 16, kT2Y = 16;            // 2-D tile; lane (x, y-group) owns 4 consecutive y

// per-marker coefficients of the spread fields (times ds / h^D)
__device__ __forceinline__ void spread_coefs(const SpreadArgs& a, int m, int D, double base, double* cf) {
  for (int c = 0; c < 8; ++c) cf[c] = 0.0;
  if (a.mode == SP_PLAIN) {
    for (int c = 0; c < 5; ++c)
      if (c < a.nf) cf[c] = a.q[(int64_t)m * a.nf + c] * base;
  } else if (a.mode == SP_STOKES) {
    const double q1 = a.q[2 * (int64_t)m], q2 = a.q[2 * (int64_t)m + 1];
    const double n1 = a.nrm[2 * (int64_t)m], n2 = a.nrm[2 * (int64_t)m + 1];
    cf[0] = 2.0 * q1 * n1 * base;
    cf[1] = (q1 * n2 + q2 * n1) * base;
    cf[2] = 2.0 * q2 * n2 * base;
    cf[3] = a.eta * q1 * base;
    cf[4] = a.eta * q2 * base;
  } else {  // SP_FDDIV: c_d = q n_d, mass in slot 3; SP_SCALAR_VEC: c_d = q n_d, mass in slot D
    const double qm = a.q[m];
    for (int d = 0; d < 3; ++d)
      if (d < D) cf[d] = qm * a.nrm[(int64_t)m * D + d] * base;
    const double mass = a.mass ? (a.eta * qm + (a.m ? a.m[m] : 0.0)) * base : 0.0;
    cf[a.mode == SP_FDDIV ? 3 : D] = mass;
  }
}

// coefficient c of marker m: the value spread_coefs leaves in cf[c] (3-D modes)
__device__ __forceinline__ double spread_coef(const SpreadArgs& a, int m, int D, double base, int c) {
  if (a.mode == SP_PLAIN) return c < a.nf ? a.q[(int64_t)m * a.nf + c] * base : 0.0;
  const double qm = a.q[m];
  if (c < D) return qm * a.nrm[(int64_t)m * D + c] * base;
  if (c == (a.mode == SP_FDDIV ? 3 : D)) return a.mass ? (a.eta * qm + (a.m ? a.m[m] : 0.0)) * base : 0.0;
  return 0.0;
}


// Candidates per wave in one pass of the 2-D spread (17 KiB of LDS per block, eight blocks per CU).
// FP64, candidates 32 (two lanes each), 16 (four), 8 (eight): the tiles of a 30-problem batch 15.5, 14.2,
// 15.9 us; 200 tiles of a 1024^2 scalar problem 6.7, 6.6, 7.0; 95 tiles with five fields 5.8, 5.4, 5.4.
template <typename T> constexpr int spread_lanes() { return sizeof(T) == 4 ? 32 : 16; }

// broadcast a lane's value to the whole wave (scalar register), any 32/64-bit type
template <typename T> __device__ __forceinline__ T bcast(T v, int lane) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
  } else {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __builtin_bit_cast(T, (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
  }
}

// ------------------------------------------------------------------ 3-D spread on the matrix cores
// A tile's spread is a sum of rank-1 tensor products, i.e. a matrix product
//   out[(y,z), x] = sum_k P[(y,z), k] Q[k, x],   k = (candidate, term),
// with Q a kernel row along x and P the matching (y,z) factor.  Finite-difference dipole field:
//   term 0: P = c_x W_y W_z,                          Q = G_x
//   term 1: P = c_y G_y W_z + c_z W_y G_z + c_m W_y W_z,  Q = W_x
// other modes (field c): P = cf_c W_y W_z, Q = W_x.  The 16 x 4 x 8 tile is two 16 x 16 blocks of
// (y,z) rows against 16 x columns; v_mfma_{f32,f64}_16x16x4 adds four k per instruction.  Operand
// layout (both precisions): lane l supplies P[l % 16][l / 16] and Q[l / 16][l % 16]; result row
// 4 (l / 16) + v (f32) or l / 16 + 4 v (f64), column l % 16.  The four waves take K-steps round
// robin and their partial tiles are added in wave order, so the result is deterministic.
template <typename T> struct Mfma;
template <> struct Mfma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};
template <> struct Mfma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};

constexpr int kSpreadWaves = 4, kSpreadCands = 64;   // launch shape of the 3-D spread
// NW waves per tile (64 NW threads) share the K-steps; SC candidates are staged per pass, four
// lanes each

template <typename T, int NF, bool FD, int NW, int SC>
__global__ __launch_bounds__(64 * NW) void k_spread3m(SpreadArgs a, const cplx<T>* __restrict__ wtab,
                                                      T* __restrict__ out) {
  using T2 = cplx<T>;
  using M = Mfma<T>;
  constexpr int kSC = SC, NTH = 64 * NW;
  constexpr int PER = (kSC * 4 + NTH - 1) / NTH;     // staging items (candidate, quarter) per thread
  constexpr int NC = FD ? 4 : NF;                    // coefficients per candidate
  constexpr int STAGE = kSC * 24 * (int)sizeof(T2) + kSC * NC * (int)sizeof(T) + kSC * 4 * (int)sizeof(int);
  constexpr int RED = NW * 512 * (int)sizeof(T);     // one field's wave partials
  __shared__ __align__(16) unsigned char smem[STAGE > RED ? STAGE : RED];
  T2(*s_w)[24] = reinterpret_cast<T2(*)[24]>(smem);                       // marker weight rows
  T(*s_c)[NC] = reinterpret_cast<T(*)[NC]>(smem + kSC * 24 * sizeof(T2));  // coefficients
  int(*s_o)[4] = reinterpret_cast<int(*)[4]>(smem + kSC * 24 * sizeof(T2) + kSC * NC * sizeof(T));
  const MarkerGeom& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int4 bt = a.busy[a.xcd ? xcd_chunk((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x];
  const int tile = bt.x;
  const int ntl = g.ntile[0] * g.ntile[1] * g.ntile[2];
  const int prob = tile / ntl, tl = tile - prob * ntl;
  const int tx = tl % g.ntile[0];
  const int ty = (tl / g.ntile[0]) % g.ntile[1];
  const int tz = tl / (g.ntile[0] * g.ntile[1]);
  const int x0 = tx * kT3X, y0 = ty * kT3Y, z0 = tz * kT3Z;
  const double hD = g.h * g.h * g.h;
  const int mx = g.n[0] - 1, my = g.n[1] - 1, mz = g.n[2] - 1;
  typename M::v4 acc[NF][2];
#pragma unroll
  for (int c = 0; c < NF; ++c) acc[c][0] = acc[c][1] = typename M::v4{0, 0, 0, 0};
  const int beg = bt.y, end = bt.z;
  constexpr int NT = FD ? 2 : 1, CPS = 4 / NT;       // terms per candidate, candidates per K-step
  const int kk = lane >> 4, i16 = lane & 15;
  const int yy = i16 & 3, zz = i16 >> 2;
  // staging: four lanes per candidate (lane quarter p loads window offset p < 3, forms the field
  // coefficients p, p + 4, ... and loads entries 6p .. 6p + 5 of the weight row), all loads of a
  // pass issued at once;
  // the next pass's marker ids are fetched while the current pass accumulates
  int m_next[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int scand = (tid + p * NTH) >> 2;
    m_next[p] = (scand < kSC && scand < end - beg) ? a.list[beg + scand] : -1;
  }
  for (int c0 = beg; c0 < end; c0 += kSC) {
    const int cnt = end - c0 < kSC ? end - c0 : kSC;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int it = tid + p * NTH, scand = it >> 2, part = it & 3;
      if (scand >= kSC) break;
      const int m = m_next[p];
      const bool live = m >= 0;
      const int mm = live ? m : 0;   // padding candidates read marker 0 and store zeros
      const T2* wrow = wtab + (int64_t)mm * 24 + 6 * part;
      T2 w6[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) w6[i] = wrow[i];
      const int o = a.s[mm * 3 + (part < 3 ? part : 0)];
      const double base = a.raw ? 1.0 : a.ds[mm] / hD;
      T cv[(NC + 3) / 4];
#pragma unroll
      for (int j = 0; j < (NC + 3) / 4; ++j)
        cv[j] = (part + 4 * j < NC) ? (T)spread_coef(a, mm, 3, base, part + 4 * j) : (T)0;
      m_next[p] = (c0 + kSC + scand < end) ? a.list[c0 + kSC + scand] : -1;
#pragma unroll
      for (int i = 0; i < 6; ++i) s_w[scand][6 * part + i] = live ? w6[i] : mk<T2>((T)0, (T)0);
      if (part < 3) s_o[scand][part] = live ? o : 6;
#pragma unroll
      for (int j = 0; j < (NC + 3) / 4; ++j)
        if (part + 4 * j < NC) s_c[scand][part + 4 * j] = live ? cv[j] : (T)0;
    }
    __syncthreads();
    const int nsteps = (cnt + CPS - 1) / CPS;
    for (int st = wave; st < nsteps; st += NW) {
      const int cand = st * CPS + kk / NT;
      // tile node -> window tap (6 and 7 hold zeros)
      const int tx_ = min((x0 + i16 - s_o[cand][0]) & mx, 6);
      const int ty_ = min((y0 + yy - s_o[cand][1]) & my, 6);
      const int tza = min((z0 + zz - s_o[cand][2]) & mz, 6);
      const int tzb = min((z0 + zz + 4 - s_o[cand][2]) & mz, 6);
      const T2 xv = s_w[cand][tx_], yv = s_w[cand][8 + ty_];
      const T2 za = s_w[cand][16 + tza], zb = s_w[cand][16 + tzb];
      if constexpr (FD) {
        const bool t0 = (kk & 1) == 0;
        const T cx = s_c[cand][0], cy = s_c[cand][1], cz = s_c[cand][2], cm = s_c[cand][3];
        const T q = t0 ? xv.y : xv.x;
        const T pyz = cy * yv.y + cm * yv.x, wy = yv.x;
        const T pa = t0 ? cx * wy * za.x : pyz * za.x + cz * wy * za.y;
        const T pb = t0 ? cx * wy * zb.x : pyz * zb.x + cz * wy * zb.y;
        acc[0][0] = M::mma(pa, q, acc[0][0]);
        acc[0][1] = M::mma(pb, q, acc[0][1]);
      } else {
        const T q = xv.x, wa = yv.x * za.x, wb = yv.x * zb.x;
#pragma unroll
        for (int c = 0; c < NF; ++c) {
          if (c < a.nf) {
            const T cf = s_c[cand][c];
            acc[c][0] = M::mma(cf * wa, q, acc[c][0]);
            acc[c][1] = M::mma(cf * wb, q, acc[c][1]);
          }
        }
      }
    }
    __syncthreads();
  }
  // fixed-order sum of the waves' partial tiles, field by field
  T* red = reinterpret_cast<T*>(smem);   // [wave][block][v][lane]
  const int64_t ntot = (int64_t)g.n[0] * g.n[1] * g.n[2];
  out += (int64_t)prob * a.nf * ntot;
#pragma unroll
  for (int c = 0; c < NF; ++c) {
    if (c >= a.nf) break;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((wave * 2 + b) * 4 + v) * 64 + lane] = acc[c][b][v];
    __syncthreads();
    for (int o = tid; o < 512; o += NTH) {
      const int b = o >> 8, v = (o >> 6) & 3, l = o & 63;
      T val = red[(b * 4 + v) * 64 + l];
#pragma unroll
      for (int w = 1; w < NW; ++w) val += red[((w * 2 + b) * 4 + v) * 64 + l];
      const int i = M::row(l, v);          // (y, z) row within the block
      const int x = l & 15, y = i & 3, z = (i >> 2) + 4 * b;
      out[c * ntot + ((int64_t)(z0 + z) * g.n[1] + (y0 + y)) * g.n[0] + x0 + x] = val;
    }
    __syncthreads();
  }
}

// The finite-difference dipole field (one output field) with the candidates' weights resolved at
// the tile's own nodes once per pass.  Each candidate's record holds G_x and W_x at the 16 x columns
// (the Q operand of terms 0 and 1) and the (W, G) pairs of its 4 y rows and 8 z planes, zero outside
// its window; the four staging lanes of a candidate fill seven of these 28 positions each, reading
// the taps the window offsets in lofs select.  A K-step then takes its operands' factors from the
// record directly: term 0 P = (c_x W_y) W_z, term 1 P = (c_y G_y + c_m W_y) W_z + (c_z W_y) G_z.
// Same products and accumulation order as k_spread3m.
template <typename T, int NW, int SC>
__global__ __launch_bounds__(64 * NW, 8) void k_spread3f(SpreadArgs a, const cplx<T>* __restrict__ wtab,
                                                      T* __restrict__ out) {
  using T2 = cplx<T>;
  using M = Mfma<T>;
  constexpr int NTH = 64 * NW;
  constexpr int PER = (SC * 4 + NTH - 1) / NTH;      // staging items (candidate, quarter) per thread
  constexpr int RS = 56;                             // record: G_x[16], W_x[16], y (W, G)[4], z (W, G)[8]
  constexpr int STAGE = SC * (RS + 4) * (int)sizeof(T);
  constexpr int RED = NW * 512 * (int)sizeof(T);
  __shared__ __align__(16) unsigned char smem[STAGE > RED ? STAGE : RED];
  T* s_r = reinterpret_cast<T*>(smem);
  T(*s_c)[4] = reinterpret_cast<T(*)[4]>(smem + SC * RS * sizeof(T));   // c_x, c_y, c_z, c_m
  const MarkerGeom& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int4 bt = a.busy[a.xcd ? xcd_chunk((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x];
  const int tile = bt.x;
  const int ntl = g.ntile[0] * g.ntile[1] * g.ntile[2];
  const int prob = tile / ntl, tl = tile - prob * ntl;
  const int tx = tl % g.ntile[0];
  const int ty = (tl / g.ntile[0]) % g.ntile[1];
  const int tz = tl / (g.ntile[0] * g.ntile[1]);
  const int x0 = tx * kT3X, y0 = ty * kT3Y, z0 = tz * kT3Z;
  const double hD = g.h * g.h * g.h;
  const int mx = g.n[0] - 1, my = g.n[1] - 1, mz = g.n[2] - 1;
  typename M::v4 acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  const int beg = bt.y, end = bt.z;
  const int i16 = lane & 15, yy = i16 & 3, zz = i16 >> 2;
  const bool t0 = ((lane >> 4) & 1) == 0;            // term of this lane's k column
  const int qoff = (t0 ? 0 : 16) + i16;
  int m_next[PER], o_next[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int scand = (tid + p * NTH) >> 2;
    const bool in = scand < SC && scand < end - beg;
    m_next[p] = in ? a.list[beg + scand] : -1;
    o_next[p] = in ? a.lofs[beg + scand] : 0;
  }
  for (int c0 = beg; c0 < end; c0 += SC) {
    const int cnt = end - c0 < SC ? end - c0 : SC;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int it = tid + p * NTH, scand = it >> 2, part = it & 3;
      if (scand >= SC) break;
      const int m = m_next[p], d = o_next[p];
      const bool live = m >= 0;
      const int mm = live ? m : 0;   // padding candidates read marker 0 and store zeros
      // lane quarter p resolves x columns p, p + 4, p + 8, p + 12, y row p and z planes p, p + 4; the
      // weight row is read at 32-bit byte offsets from the launch-uniform table
      const unsigned wrow = (unsigned)mm * 24u * (unsigned)sizeof(T2);
      const int dx = d & 1023, dy = (d >> 10) & 1023, dz = (d >> 20) & 1023;
      unsigned slot[7];
#pragma unroll
      for (int i = 0; i < 4; ++i) slot[i] = (unsigned)((part + 4 * i - dx) & mx);
      slot[4] = (unsigned)((part - dy) & my);
      slot[5] = (unsigned)((part - dz) & mz);
      slot[6] = (unsigned)((part + 4 - dz) & mz);
      T2 e[7];
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        const unsigned base = i < 4 ? 0u : (i == 4 ? 8u : 16u);
        const unsigned sl = base + (slot[i] < 6u ? slot[i] : 6u);   // taps 6 and 7 of a row are zero
        e[i] = *reinterpret_cast<const T2*>(reinterpret_cast<const char*>(wtab) + (wrow + sl * (unsigned)sizeof(T2)));
      }
      const T cv = (T)spread_coef(a, mm, 3, a.raw ? 1.0 : a.ds[mm] / hD, part);
      const bool more = c0 + SC + scand < end;
      m_next[p] = more ? a.list[c0 + SC + scand] : -1;
      o_next[p] = more ? a.lofs[c0 + SC + scand] : 0;
      T* r = s_r + scand * RS;
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        const T w = live ? e[i].x : (T)0, gd = live ? e[i].y : (T)0;
        if (i < 4) {            // x column: G_x (term 0), W_x (term 1)
          r[part + 4 * i] = gd;
          r[16 + part + 4 * i] = w;
        } else {                // y row / z plane: (W, G)
          const int o = i == 4 ? 32 + 2 * part : (i == 5 ? 40 + 2 * part : 48 + 2 * part);
          r[o] = w;
          r[o + 1] = gd;
        }
      }
      s_c[scand][part] = live ? cv : (T)0;
    }
    __syncthreads();
    const int nsteps = (cnt + 1) >> 1;
    for (int st = wave; st < nsteps; st += NW) {
      const int cand = 2 * st + (lane >> 5);
      const T* r = s_r + cand * RS;
      const T q = r[qoff];
      const T2 yv = *reinterpret_cast<const T2*>(r + 32 + 2 * yy);
      const T2 za = *reinterpret_cast<const T2*>(r + 40 + 2 * zz);
      const T2 zb = *reinterpret_cast<const T2*>(r + 48 + 2 * zz);
      const T cx = s_c[cand][0], cy = s_c[cand][1], cz = s_c[cand][2], cm = s_c[cand][3];
      const T u = t0 ? cx * yv.x : cy * yv.y + cm * yv.x;
      const T v = t0 ? (T)0 : cz * yv.x;
      acc0 = M::mma(u * za.x + v * za.y, q, acc0);
      acc1 = M::mma(u * zb.x + v * zb.y, q, acc1);
    }
    __syncthreads();
  }
  // fixed-order sum of the waves' partial tiles
  T* red = reinterpret_cast<T*>(smem);   // [wave][block][v][lane]
  const int64_t ntot = (int64_t)g.n[0] * g.n[1] * g.n[2];
  out += (int64_t)prob * ntot;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    red[((wave * 2 + 0) * 4 + v) * 64 + lane] = acc0[v];
    red[((wave * 2 + 1) * 4 + v) * 64 + lane] = acc1[v];
  }
  __syncthreads();
  for (int o = tid; o < 512; o += NTH) {
    const int b = o >> 8, v = (o >> 6) & 3, l = o & 63;
    T val = red[(b * 4 + v) * 64 + l];
#pragma unroll
    for (int w = 1; w < NW; ++w) val += red[((w * 2 + b) * 4 + v) * 64 + l];
    const int i = M::row(l, v);
    const int x = l & 15, y = i & 3, z = (i >> 2) + 4 * b;
    out[((int64_t)(z0 + z) * g.n[1] + (y0 + y)) * g.n[0] + x0 + x] = val;
  }
}

// 2-D: a tile of TX x TY nodes (TX TY = 256, TY = 4 (64 / TX) rows); lane (x, y-group) owns
// y = 4 yg + j' (j' < 4).  Wave w takes candidates w, w + 4, ... of the tile's list, LW at a time: 64 / LW
// lanes copy a candidate's x and y weight rows to LDS, the first of them keeps its window start and
// coefficients, which are broadcast; a node's taps are picked by index.  The rows are copied as they are,
// so everything a candidate needs is loaded at once behind its list entry (which is read a round ahead): the
// launch is a chain of dependent loads (tile, list entry, marker), a few candidates' work per wave, and the
// sum over the waves.  (The y rows had been aligned to the tile as they were staged, one more dependent load
// and 48 KiB of LDS in double, then copied by one lane per candidate, sixteen loads each and 34 KiB: five
// Stokes fields on 95 tiles 6.7 -> 5.4 us with several lanes, on the 774 tiles of a 4096^2 array 9.7 -> 7.8 us,
// the tiles of a 30-problem batch 22.2 -> 18.2 -> 14.2 us.)
// s_w is the caller's LDS, [4][LW][kSpreadRow] (W, G) pairs: a candidate's x taps at 0 .. 5, its y taps at
// 9 .. 14, zeros between and after, so that a lane's four y nodes are four neighbouring pairs of one clamped
// index.  On crowded tiles a candidate's instructions are what counts: 24,000 markers on a ring of a 512^2
// grid (28 to a cell's length) took 57 us in double and 44 in single precision with aligned rows, 54 and 49
// with an index for each y node, and take 43 and 34 with one index and two candidates at a time; 1,600
// markers 8.8 and 8.2, 8.0 and 8.0, 7.5 and 7.2.  Single precision with several fields gains nothing from
// the pairs and takes its candidates one by one.
constexpr int kSpreadRow = 19;
template <typename T, int NF, int TX>
__device__ __forceinline__ void spread2_tile(const SpreadArgs& a, const cplx<T>* __restrict__ wtab, T* __restrict__ out,
                                             const int4 bt, cplx<T> (*s_w)[spread_lanes<T>()][kSpreadRow]) {
  using T2 = cplx<T>;
  constexpr int LW = spread_lanes<T>();
  constexpr int TY = 256 / TX;
  static_assert(TX * TY == 256 && TX >= 4 && TX <= 64, "2-D tile of 256 nodes, 64 lanes of 4 rows");
  const MarkerGeom& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = bt.x;
  const int ntl = g.ntile[0] * g.ntile[1];
  const int prob = tile / ntl, tl = tile - prob * ntl;
  const int tx = tl % g.ntile[0];
  const int ty = tl / g.ntile[0];
  const int x0 = tx * TX, y0 = ty * TY;
  const int lx = lane % TX, yg = lane / TX;
  const int mx = g.n[0] - 1, my = g.n[1] - 1;
  const bool fddiv = NF == 1 && a.mode == SP_FDDIV;
  T acc[4][NF];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int c = 0; c < NF; ++c) acc[j][c] = 0;
  const int beg = bt.y, end = bt.z;
  const double hD = g.h * g.h;
  constexpr int NP = 64 / LW, NW = 16 / NP;   // lanes per candidate, weights copied by each
  const int cd = lane % LW, part = lane / LW;
  static_assert(NW <= 8, "a lane copies taps of one axis");
  T2* mine = &s_w[wave][cd][part * NW + (part * NW >= 8 ? 1 : 0)];
  if (part == 0) s_w[wave][cd][8] = mk<T2>((T)0, (T)0);
  if (part == 1) s_w[wave][cd][17] = s_w[wave][cd][18] = mk<T2>((T)0, (T)0);
  const int at = beg + 4 * cd + wave;
  int m_next = at < end ? a.list[at] : -1;   // a list entry is read a round ahead
  for (int c0 = beg; c0 < end; c0 += 4 * LW) {
    const int left = end - c0 - wave;
    const int cnt = left <= 0 ? 0 : ((left + 3) / 4 < LW ? (left + 3) / 4 : LW);
    int sx = 0, sy = 0;
    T cf[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) cf[c] = 0;
    const int m = m_next, an = c0 + 4 * (LW + cd) + wave;
    m_next = an < end ? a.list[an] : -1;
    if (m >= 0) {
      const T2* row = wtab + (int64_t)m * 24 + part * NW;
      T2 w[NW];
#pragma unroll
      for (int t = 0; t < NW; ++t) w[t] = row[t];
      sx = a.s[m * 3 + 0];
      sy = a.s[m * 3 + 1];
      double c8[8];
      spread_coefs(a, m, 2, a.raw ? 1.0 : a.ds[m] / hD, c8);
#pragma unroll
      for (int c = 0; c < 5; ++c) cf[c] = (T)c8[c];
#pragma unroll
      for (int t = 0; t < NW; ++t) mine[t] = w[t];
    }
    // (each wave reads its own rows only)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    auto taps = [&](int j, T2& xv, T2 (&yv)[4]) {
      // node - window start: taps 0 .. 5 of x, rows -3 .. 5 of the lane's first y node
      xv = s_w[wave][j][min((x0 + lx - bcast(sx, j)) & mx, 6)];
      const T2* yp = &s_w[wave][j][6 + min((y0 + 4 * yg + 3 - bcast(sy, j)) & my, 9)];
#pragma unroll
      for (int q = 0; q < 4; ++q) yv[q] = yp[q];
    };
    auto add = [&](int j, const T2& xv, const T2 (&yv)[4]) {
      if (fddiv) {
        // v = c_x G_x W_y + c_y W_x G_y + c_mass W_x W_y
        const T ax = bcast(cf[0], j) * xv.y + bcast(cf[3], j) * xv.x, ay = bcast(cf[1], j) * xv.x;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q][0] += ax * yv[q].x + ay * yv[q].y;
      } else {
#pragma unroll
        for (int c = 0; c < NF; ++c) {
          if (c < a.nf) {
            const T cx = bcast(cf[c], j) * xv.x;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q][c] += cx * yv[q].x;
          }
        }
      }
    };
    int j = 0;
    if constexpr (NF == 1 || sizeof(T) == 8) {   // two at a time: the second's taps arrive while the first is summed
      for (; j + 1 < cnt; j += 2) {
        T2 xa, ya[4], xb, yb[4];
        taps(j, xa, ya);
        taps(j + 1, xb, yb);
        __builtin_amdgcn_sched_barrier(0);
        add(j, xa, ya);
        add(j + 1, xb, yb);
      }
    }
    for (; j < cnt; ++j) {
      T2 xa, ya[4];
      taps(j, xa, ya);
      add(j, xa, ya);
    }
    __builtin_amdgcn_wave_barrier();
  }
  // sum of the waves' parts in wave order, as many fields at a time as the LDS holds
  T* red = reinterpret_cast<T*>(&s_w[0][0][0]);
  constexpr int FR = 4 * LW * 16 * 2 / 1024;   // fields of [4][4][64] values
  static_assert(FR >= 1, "spread: LDS holds a field's partial tiles");
  const int64_t ntot = (int64_t)g.n[0] * g.n[1];
  out += (int64_t)prob * a.nf * ntot;
  const int q = tid >> 6, l = lane;   // 256 tile nodes, one per thread: l (x, y-group), q: y within the group
  T* dst = out + (int64_t)(y0 + 4 * (l / TX) + q) * g.n[0] + x0 + l % TX;
#pragma unroll
  for (int c0 = 0; c0 < NF; c0 += FR) {
    if (c0 >= a.nf) break;
    __syncthreads();
#pragma unroll
    for (int c = c0; c < NF && c < c0 + FR; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) red[((c - c0) * 16 + wave * 4 + k) * 64 + lane] = acc[k][c];
    __syncthreads();
#pragma unroll
    for (int c = c0; c < NF && c < c0 + FR; ++c) {
      if (c >= a.nf) break;
      const T* r = red + (c - c0) * 1024 + l;
      dst[c * ntot] = ((r[q * 64] + r[(4 + q) * 64]) + r[(8 + q) * 64]) + r[(12 + q) * 64];
    }
  }
}

template <typename T, int NF>
__global__ __launch_bounds__(256) void k_spread2(SpreadArgs a, const cplx<T>* __restrict__ wtab, T* __restrict__ out) {
  __shared__ cplx<T> s_w[4][spread_lanes<T>()][kSpreadRow];
  spread2_tile<T, NF, kT2X>(a, wtab, out, a.busy[blockIdx.x], s_w);
}

// The spread of several grid groups (a batch) in one persistent launch over a single work list,
// items[k] = (group, busy-tile index), ordered by decreasing candidate count across all groups:
// workgroup b takes items b, b + G, b + 2 G, ... (G workgroups), so the longest tiles go first and
// every workgroup ends with short ones.  (A shared atomic counter was measured slower: 4,500 tiles
// serialise on one address.)  Each group has its own arguments, weight table, output fields and
// tile width (16, 32 or 64 nodes along x); its densities are qbase + qoff.
template <typename T>
__global__ __launch_bounds__(256) void k_spread2_queue(const SpreadGroup* __restrict__ gd, const int2* __restrict__ items,
                                                       int nitems, const double* __restrict__ qbase) {
  __shared__ cplx<T> s_w[4][spread_lanes<T>()][kSpreadRow];
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int2 gi = items[it];
    const int gsel = __builtin_amdgcn_readfirstlane(gi.x);
    SpreadArgs a = gd[gsel].a;
    a.q = qbase + gd[gsel].qoff;
    const int4 bt = a.busy[gi.y];
    const cplx<T>* wt = reinterpret_cast<const cplx<T>*>(gd[gsel].wtab);
    T* out = reinterpret_cast<T*>(gd[gsel].out);
    const int tw = gd[gsel].tx;
    if (it != (int)blockIdx.x) __syncthreads();   // the last tile's sums are read
    if (tw == 32) spread2_tile<T, 1, 32>(a, wt, out, bt, s_w);
    else if (tw == 64) spread2_tile<T, 1, 64>(a, wt, out, bt, s_w);
    else spread2_tile<T, 1, 16>(a, wt, out, bt, s_w);
  }
}

// ------------------------------------------------------------------ interpolation
// Workgroup c of the border workgroups behind the nmain of an interpolation (BorderArgs)
__device__ __forceinline__ void border_block(const BorderArgs& bd, int c) {
  __shared__ double red[4];
  double s = 0.0;
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < bd.n; i += 256) s += (bd.w ? bd.w[i] : 1.0) * bd.q[i * bd.nq + c];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) bd.out[c] = bd.scale * (((red[0] + red[1]) + red[2]) + red[3]);
}

// y of marker i from its interpolated adjoint fields G (see k_adj_combine)
__device__ __forceinline__ void adj_marker(const AdjArgs& ad, int64_t i, int ng, const double* G, double* __restrict__ y) {
  const double w = ad.hDinv * ad.ds[i];
  if (!ad.stokes) {
    double s = 0.0;
    if (ad.dim == 2) s = ad.nrm[2 * i] * G[0] + ad.nrm[2 * i + 1] * G[1] - (ng > 2 ? ad.eta * G[2] : 0.0);
    else
      s = ad.nrm[3 * i] * G[0] + ad.nrm[3 * i + 1] * G[1] + ad.nrm[3 * i + 2] * G[2] - (ng > 3 ? ad.eta * G[3] : 0.0);
    double v = w * s;
    if (ad.p) v += ad.b * ad.p[i];
    if (ad.pu) v += ad.eta * ad.ds[i] * ad.pu[0];
    y[i] = v;
    return;
  }
  const double n1 = ad.nrm[2 * i], n2 = ad.nrm[2 * i + 1];
  double s1 = 2.0 * n1 * G[0] + n2 * G[1];
  double s2 = n1 * G[1] + 2.0 * n2 * G[2];
  if (ng > 3) {
    s1 += ad.eta * G[3];
    s2 += ad.eta * G[4];
  }
  double v1 = w * s1, v2 = w * s2;
  if (ad.p) {
    v1 += ad.b * ad.p[2 * i];
    v2 += ad.b * ad.p[2 * i + 1];
  }
  if (ad.pu) {
    v1 += ad.eta * ad.ds[i] * ad.pu[0];
    v2 += ad.eta * ad.ds[i] * ad.pu[1];
  }
  y[2 * i] = v1;
  y[2 * i + 1] = v2;
}

template <typename T, int D, int K>
__global__ __launch_bounds__(256) void k_interp(InterpArgs a, const T* __restrict__ u, double* __restrict__ out,
                                                int nmain, BorderArgs bd) {
  if ((int)blockIdx.x >= nmain) {
    border_block(bd, (int)blockIdx.x - nmain);
    return;
  }
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n_ib) return;
  const MarkerGeom& g = a.g;
  constexpr int T0 = (K == 4) ? 1 : 0;
  T w[3][K];
  int ix[3][K];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double* row = a.wt + (i * 3 + d) * 12;
    const int s = a.s[i * 3 + d];
#pragma unroll
    for (int t = 0; t < K; ++t) {
      w[d][t] = (d < D) ? (T)row[t + T0] : (T)(t == 0);
      ix[d][t] = (d < D) ? ((s + t + T0) & (g.n[d] - 1)) : 0;
    }
  }
  const int64_t ntot = (int64_t)g.n[0] * g.n[1] * (D == 3 ? g.n[2] : 1);
  if (a.pid) u += (int64_t)a.pid[i] * a.nf * ntot;
  for (int c = 0; c < a.nf; ++c) {
    const T* uc = u + c * ntot;
    T acc = 0;
    constexpr int KZ = (D == 3) ? K : 1;
#pragma unroll
    for (int tz = 0; tz < KZ; ++tz) {
#pragma unroll
      for (int ty = 0; ty < K; ++ty) {
        const T wyz = w[1][ty] * (D == 3 ? w[2][tz] : (T)1);
        const int64_t row = ((int64_t)(D == 3 ? ix[2][tz] : 0) * g.n[1] + ix[1][ty]) * g.n[0];
        T rs = 0;
#pragma unroll
        for (int tx = 0; tx < K; ++tx) rs += uc[row + ix[0][tx]] * w[0][tx];
        acc += rs * wyz;
      }
    }
    double v = a.a * (double)acc;
    if (a.x) v += a.b * a.x[i * a.nf + c];
    if (a.ub) v += a.ub[c];
    out[i * a.nf + c] = v;
  }
}

// 4-point kernels: a group of RL = 4^(D-1) lanes per marker, lane r of the group sums the 4 x-taps of
// stencil row r of each of the nf <= NF fields (every field's loads issued before the first sum); the
// row sums are reduced across the group by a fixed butterfly (deterministic).  Workgroup b of nmain; the
// group's lane 0 calls done(i, v) with marker i's sums.
template <typename T, int D, int NF, typename F>
__device__ __forceinline__ void interp4_block(const InterpArgs& a, const cplx<T>* __restrict__ wtab,
                                              const T* __restrict__ u, int b, int nmain, F&& done) {
  constexpr int RL = (D == 3) ? 16 : 4;
  // XCD-contiguous marker ranges: markers close in index share grid lines, so they share an L2
  const int64_t gid = (int64_t)xcd_chunk(b, nmain) * 256 + threadIdx.x;
  const int64_t i = gid / RL;
  const int r = (int)(gid % RL);
  const bool valid = i < a.n_ib;
  const int64_t im = valid ? i : 0;
  const MarkerGeom& g = a.g;
  const cplx<T>* row = wtab + im * 24;       // axis d taps at row[d*8 + t], t = 1..4 non-zero
  const int sx = a.s[im * 3 + 0], sy = a.s[im * 3 + 1], sz = a.s[im * 3 + 2];
  const int ty = r & 3, tz = r >> 2;         // stencil row (y tap, z tap)
  const T wyz = row[8 + 1 + ty].x * (D == 3 ? row[16 + 1 + tz].x : (T)1);
  const int64_t base = ((int64_t)(D == 3 ? ((sz + 1 + tz) & (g.n[2] - 1)) : 0) * g.n[1] +
                        ((sy + 1 + ty) & (g.n[1] - 1))) * g.n[0];
  int ix[4];
  T wx[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    ix[t] = (sx + 1 + t) & (g.n[0] - 1);
    wx[t] = row[1 + t].x;
  }
  const int64_t ntot = (int64_t)g.n[0] * g.n[1] * (D == 3 ? g.n[2] : 1);
  if (a.pid) u += (int64_t)a.pid[im] * a.nf * ntot;
  T v[NF];
#pragma unroll
  for (int c = 0; c < NF; ++c) {
    const T* uc = u + (NF > 1 && c < a.nf ? c : 0) * ntot + base;
    v[c] = ((uc[ix[0]] * wx[0] + uc[ix[1]] * wx[1]) + uc[ix[2]] * wx[2] + uc[ix[3]] * wx[3]) * wyz;
  }
#pragma unroll
  for (int c = 0; c < NF; ++c)
#pragma unroll
    for (int off = 1; off < RL; off <<= 1) v[c] += __shfl_xor(v[c], off, RL);
  if (valid && r == 0) done(i, v);
}
template <typename T, int NF> __device__ __forceinline__ void interp4_store(const InterpArgs& a, int64_t i, const T (&v)[NF],
                                                                            double* __restrict__ out) {
#pragma unroll
  for (int c = 0; c < NF; ++c) {
    if (NF == 1 || c < a.nf) {
      double o = a.a * (double)v[c];
      if (a.x) o += a.b * a.x[i * a.nf + c];
      if (a.ub) o += a.ub[c];
      out[i * a.nf + c] = o;
    }
  }
}

template <typename T, int D, int NF>
__global__ __launch_bounds__(256) void k_interp4(InterpArgs a, const cplx<T>* __restrict__ wtab, const T* __restrict__ u,
                                                 double* __restrict__ out) {
  interp4_block<T, D, NF>(a, wtab, u, blockIdx.x, gridDim.x,
                          [&](int64_t i, const T (&v)[NF]) { interp4_store<T, NF>(a, i, v, out); });
}
// With border sums in further workgroups, a kernel of its own: the branch in front cost the others half a
// microsecond (18,500 markers in 3-D).  Latency-bound: with the border sums and the adjoint's combination in
// the interpolation's launch, a 1024^2 Stokes apply went from 56.3 to 50.6 us and a 512^2 Stokes adjoint step
// lost three launches of 1.8 to 4.6 us.
template <typename T, int D, int NF>
__global__ __launch_bounds__(256) void k_interp4_border(InterpArgs a, const cplx<T>* __restrict__ wtab,
                                                        const T* __restrict__ u, double* __restrict__ out, int nmain,
                                                        BorderArgs bd) {
  if ((int)blockIdx.x >= nmain) {
    border_block(bd, (int)blockIdx.x - nmain);
    return;
  }
  interp4_block<T, D, NF>(a, wtab, u, blockIdx.x, nmain,
                          [&](int64_t i, const T (&v)[NF]) { interp4_store<T, NF>(a, i, v, out); });
}
// The fields combined into the transposed operator's marker values instead of stored
template <typename T, int D>
__global__ __launch_bounds__(256) void k_interp4_adj(InterpArgs a, AdjArgs ad, const cplx<T>* __restrict__ wtab,
                                                     const T* __restrict__ u, double* __restrict__ out, int nmain,
                                                     BorderArgs bd) {
  if ((int)blockIdx.x >= nmain) {
    border_block(bd, (int)blockIdx.x - nmain);
    return;
  }
  interp4_block<T, D, 5>(a, wtab, u, blockIdx.x, nmain, [&](int64_t i, const T (&v)[5]) {
    double G[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) G[c] = (double)v[c];
    adj_marker(ad, i, a.nf, G, out);
  });
}

// The interpolation (4-point kernels, 2-D) of several grid groups in one launch: marker i of the
// concatenation belongs to the group g with m0[g] <= i < m0[g + 1] (gd[g].m0); it reads that group's
// fields and weight table and writes out[i] = a S*u + b x[i] (one field per marker).
template <typename T>
__global__ __launch_bounds__(256) void k_interp4_groups(const InterpGroup* __restrict__ gd, int ng, int64_t ntot_m,
                                                        const double* __restrict__ xbase, double* __restrict__ out) {
  constexpr int RL = 4;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = gid / RL;
  const int r = (int)(gid % RL);
  const bool valid = i < ntot_m;
  const int64_t ic = valid ? i : 0;
  int gsel = 0;
  while (gsel + 1 < ng && ic >= gd[gsel + 1].m0) ++gsel;
  const InterpGroup& G = gd[gsel];
  const MarkerGeom& g = G.a.g;
  const int64_t im = ic - G.m0;
  const cplx<T>* row = reinterpret_cast<const cplx<T>*>(G.wtab) + im * 24;
  const int sx = G.a.s[im * 3 + 0], sy = G.a.s[im * 3 + 1];
  const int ty = r & 3;
  const T wyz = row[8 + 1 + ty].x;
  const int64_t base = (int64_t)((sy + 1 + ty) & (g.n[1] - 1)) * g.n[0];
  int ix[4];
  T wx[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    ix[t] = (sx + 1 + t) & (g.n[0] - 1);
    wx[t] = row[1 + t].x;
  }
  const int64_t ntot = (int64_t)g.n[0] * g.n[1];
  const T* uc = reinterpret_cast<const T*>(G.u) + (int64_t)G.a.pid[im] * ntot + base;
  T v = ((uc[ix[0]] * wx[0] + uc[ix[1]] * wx[1]) + uc[ix[2]] * wx[2] + uc[ix[3]] * wx[3]) * wyz;
#pragma unroll
  for (int off = 1; off < RL; off <<= 1) v += __shfl_xor(v, off, RL);
  if (valid && r == 0) {
    double o = G.a.a * (double)v;
    if (xbase) o += G.a.b * xbase[i];
    out[i] = o;
  }
}

// Transpose of the fused FD divergence spread (SP_FDDIV), for the scalar transposed operator with
// centred differences.  Per marker, over the 6-node window (G_d spans all 6 taps, W the inner 4),
//   v_i = sum_y w(y) [sum_d n_id G_d(y) prod_{e != d} W_e(y) + eta prod_e W_e(y)]
// and, since Phi D_d = -(the G_d-weighted interpolation) when D_d is the centred difference,
//   y_i = -h^-D ds_i v_i + b p_i + eta ds_i pu        (p = a.x, b = a.b; pu: the ubar entries or null)
// which equals h^-D ds_i (sum_d n_id Phi D_d w - eta Phi w) + b p_i + eta ds_i pu.
// 3-D: 32 lanes per marker, one per (y, z) stencil row of the 6 x 6 window less its 4 corners
// (W_y and W_z both vanish there); 2-D: 8 lanes, the first 6 one per y row.  Each lane reads the 6
// x taps of its row against A G_x + B W_x; the row sums are reduced by a fixed butterfly.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_interp_div(InterpArgs a, const cplx<T>* __restrict__ wtab,
                                                    const T* __restrict__ u, const double* __restrict__ nrm,
                                                    const double* __restrict__ ds, double eta, double hDinv,
                                                    const double* __restrict__ pu, double* __restrict__ y, int nmain,
                                                    BorderArgs bd) {
  constexpr int RL = (D == 3) ? 32 : 8;
  if ((int)blockIdx.x >= nmain) {
    border_block(bd, (int)blockIdx.x - nmain);
    return;
  }
  const int64_t gid = (int64_t)xcd_chunk(blockIdx.x, nmain) * blockDim.x + threadIdx.x;
  const int64_t i = gid / RL;
  const int r = (int)(gid % RL);
  const bool valid = i < a.n_ib;
  const int64_t im = valid ? i : 0;
  const MarkerGeom& g = a.g;
  const cplx<T>* row = wtab + im * 24;       // axis d taps at row[d*8 + t], t < 6
  int ty = r, tz = 0;
  if (D == 3) {
    const int k = r + 1 + (r >= 4 ? 1 : 0) + (r >= 28 ? 1 : 0);   // skips k = 0, 5, 30, 35
    ty = k % 6;
    tz = k / 6;
  }
  const bool live = D == 3 || r < 6;
  const cplx<T> py = row[8 + (live ? ty : 0)];
  const cplx<T> pz = D == 3 ? row[16 + tz] : mk<cplx<T>>((T)1, (T)0);
  const T n0 = (T)nrm[im * D], n1 = (T)nrm[im * D + 1], n2 = D == 3 ? (T)nrm[im * D + 2] : (T)0;
  const T A = n0 * py.x * pz.x;
  const T B = n1 * py.y * pz.x + n2 * py.x * pz.y + (T)eta * py.x * pz.x;
  const int sx = a.s[im * 3 + 0], sy = a.s[im * 3 + 1], sz = a.s[im * 3 + 2];
  const int64_t base = ((int64_t)(D == 3 ? ((sz + tz) & (g.n[2] - 1)) : 0) * g.n[1] + ((sy + ty) & (g.n[1] - 1))) *
                       g.n[0];
  T v = 0;
  if (live) {
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const cplx<T> px = row[t];
      v += u[base + ((sx + t) & (g.n[0] - 1))] * (A * px.y + B * px.x);
    }
  }
#pragma unroll
  for (int off = 1; off < RL; off <<= 1) v += __shfl_xor(v, off, RL);
  if (valid && r == 0) {
    double o = -hDinv * ds[i] * (double)v;
    if (a.x) o += a.b * a.x[i];
    if (pu) o += eta * ds[i] * pu[0];
    y[i] = o;
  }
}

// ------------------------------------------------------------------ active rows
// Rows y of plane z that a marker's 6-node window meets: [s_y, s_y + 5] for z in [s_z, s_z + 5]
// (mod n); a window that wraps around y marks the whole plane.
__global__ void k_rows_init(int* __restrict__ lo, int* __restrict__ hi, int nplanes, int ny,
                            unsigned long long* __restrict__ count) {
  const int z = blockIdx.x * blockDim.x + threadIdx.x;
  if (z == 0) *count = 0;
  if (z < nplanes) {
    lo[z] = ny;
    hi[z] = -1;
  }
}

// per-block limits in LDS first (many markers share a plane), then one global update per touched plane
__global__ __launch_bounds__(256) void k_rows_mark(MarkerGeom g, int64_t n_ib, const int* __restrict__ s,
                                                   int* __restrict__ lo, int* __restrict__ hi) {
  extern __shared__ int sm[];
  const int ny = g.n[1];
  const int nz = g.dim == 3 ? g.n[2] : 1;
  int* slo = sm;
  int* shi = sm + nz;
  for (int z = threadIdx.x; z < nz; z += blockDim.x) {
    slo[z] = ny;
    shi[z] = -1;
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_ib) {
    const int sy = s[i * 3 + 1];
    const int ylo = sy + 5 < ny ? sy : 0;
    const int yhi = sy + 5 < ny ? sy + 5 : ny - 1;
    const int nw = g.dim == 3 ? 6 : 1;
    for (int t = 0; t < nw; ++t) {
      const int z = g.dim == 3 ? (s[i * 3 + 2] + t) & (nz - 1) : 0;
      atomicMin(&slo[z], ylo);
      atomicMax(&shi[z], yhi);
    }
  }
  __syncthreads();
  for (int z = threadIdx.x; z < nz; z += blockDim.x) {
    if (shi[z] >= 0) {
      atomicMin(&lo[z], slo[z]);
      atomicMax(&hi[z], shi[z]);
    }
  }
}

// Per-plane row counts, their scan, and the (lo, hi) pairs used by the y-pass masks; one block of 1024
// threads.  host (pinned): the number of busy tiles, of active rows, and the pairs, for the caller to
// read after a wait on the stream.
__global__ __launch_bounds__(1024) void k_rows_count(const int* __restrict__ lo, const int* __restrict__ hi, int nplanes,
                                                     int* __restrict__ cnt, int* __restrict__ off, int2* __restrict__ lim,
                                                     const int* __restrict__ nbusy, int* __restrict__ host) {
  __shared__ int s_w[16];
  int carry = 0;
  for (int base = 0; base < nplanes; base += 1024) {
    const int z = base + (int)threadIdx.x;
    int2 l = make_int2(1, 0);
    if (z < nplanes && hi[z] >= lo[z]) l = make_int2(lo[z], hi[z]);
    const int c = l.y - l.x + 1;
    int tot;
    const int o = carry + block_scan(c, s_w, tot);
    if (z < nplanes) {
      cnt[z] = c;
      off[z] = o;
      lim[z] = l;
      host[2 + 2 * z] = l.x;
      host[3 + 2 * z] = l.y;
    }
    carry += tot;
  }
  if (threadIdx.x == 0) {
    off[nplanes] = carry;
    host[0] = *nbusy;
    host[1] = carry;
  }
}

__global__ void k_rows_list(const int* __restrict__ lo, const int* __restrict__ cnt, const int* __restrict__ off,
                            int nplanes, int ny, int* __restrict__ rows) {
  const int z = blockIdx.x;
  if (z >= nplanes) return;
  for (int k = threadIdx.x; k < cnt[z]; k += blockDim.x) rows[off[z] + k] = z * ny + lo[z] + k;
}


// ------------------------------------------------------------------ kernel-derivative gather
// Sixteen lanes per marker over its K^D window (K = 4: taps 1..4 of the 6-node window; K = 6: all), in
// double: out[i][e] = sum_x F_i(x) (-phi'(r_e)/h) prod_{d != e} phi(r_d), r_d = (x_d - X_id)/h.  A lane
// takes a row of the window (in 2-D a node), its weights staged in LDS by the whole block.  Bound by the
// latency of scattered loads, so lanes: with one thread per marker the 64 nodes x fields of a window were
// one chain on a few waves (18,500 markers, 3-D, FP64: 94 us on 73 workgroups, now 14; 1,024 markers,
// 2-D, 5 fields: 41 us, now 8).
constexpr int kGatherLanes = 16;
template <typename T, int D, int K>
__global__ __launch_bounds__(256) void k_gather_dx(GatherArgs a) {
  constexpr int LN = kGatherLanes, MPB = 256 / LN, T0 = (K == 4) ? 1 : 0, NF = 8;
  __shared__ double s_w[MPB][3][K], s_dw[MPB][3][K], s_cf[MPB][NF];
  __shared__ int s_ix[MPB][3][K];
  const MarkerGeom& g = a.g;
  const int64_t i0 = (int64_t)blockIdx.x * MPB;
  for (int t = threadIdx.x; t < MPB * 3 * K; t += 256) {
    const int m = t / (3 * K), d = t / K % 3, k = t % K;
    const int64_t i = i0 + m;
    double w = (D == 2 && d == 2) ? 1.0 : 0.0, dw = 0.0;
    int ix = 0;
    if (d < D && i < a.n_ib) {
      const double r = (double)(k + T0 - 2) - a.f[i * 3 + d];
      w = phi_eval(a.kernel, r);
      dw = -dphi_eval(a.kernel, r) / g.h;
      ix = (a.s[i * 3 + d] + k + T0) & (g.n[d] - 1);
    }
    s_w[m][d][k] = w;
    s_dw[m][d][k] = dw;
    s_ix[m][d][k] = ix;
  }
  if (threadIdx.x < MPB * NF) {
    const int m = threadIdx.x / NF, k = threadIdx.x % NF;
    s_cf[m][k] = (k < a.nfield && i0 + m < a.n_ib) ? a.coef[(i0 + m) * a.nfield + k] : 0.0;
  }
  __syncthreads();
  const int m = threadIdx.x / LN, lane = threadIdx.x % LN;
  constexpr int NX = D == 3 ? K : 1;   // nodes of a lane's item
  double acc[3] = {0.0, 0.0, 0.0};
  if (i0 + m < a.n_ib) {
    for (int q = lane; q < K * K; q += LN) {
      const int t1 = q / K, t0 = q % K;
      // item q: the x row at (y, z) = (t0, t1) in 3-D, the node (x, y) = (t0, t1) in 2-D
      const int64_t row = D == 3 ? ((int64_t)s_ix[m][2][t1] * g.n[1] + s_ix[m][1][t0]) * g.n[0]
                                 : (int64_t)s_ix[m][1][t1] * g.n[0] + s_ix[m][0][t0];
      double F[NX];
#pragma unroll
      for (int x = 0; x < NX; ++x) F[x] = 0.0;
      for (int k0 = 0; k0 < a.nfield; k0 += 4) {
        T v[4][NX];
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // fields beyond the last: loaded again and not used
          const T* fld = static_cast<const T*>(a.field[k0 + k < a.nfield ? k0 + k : 0]) + row;
#pragma unroll
          for (int x = 0; x < NX; ++x) v[k][x] = fld[D == 3 ? s_ix[m][0][x] : 0];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k0 + k >= a.nfield) break;
#pragma unroll
          for (int x = 0; x < NX; ++x) F[x] += s_cf[m][k0 + k] * (double)v[k][x];
        }
      }
      if constexpr (D == 3) {
        double fw = 0.0, fd = 0.0;
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          fw += F[x] * s_w[m][0][x];
          fd += F[x] * s_dw[m][0][x];
        }
        acc[0] += fd * s_w[m][1][t0] * s_w[m][2][t1];
        acc[1] += fw * s_dw[m][1][t0] * s_w[m][2][t1];
        acc[2] += fw * s_w[m][1][t0] * s_dw[m][2][t1];
      } else {
        acc[0] += F[0] * s_dw[m][0][t0] * s_w[m][1][t1];
        acc[1] += F[0] * s_w[m][0][t0] * s_dw[m][1][t1];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < D; ++e) {
    for (int o = LN / 2; o > 0; o >>= 1) acc[e] += __shfl_xor(acc[e], o);
  }
  if (i0 + m < a.n_ib && lane == 0) {
#pragma unroll
    for (int e = 0; e < D; ++e) a.out[(i0 + m) * D + e] = acc[e];
  }
}

// ------------------------------------------------------------------ grid elementwise
template <typename T>
__global__ void k_axpby(T* __restrict__ y, double a, const T* __restrict__ x, double b, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    y[e] = (T)(a * (double)x[e] + b * (double)y[e]);
}

template <typename S, typename D>
__global__ void k_convert(const S* __restrict__ x, D* __restrict__ y, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    y[e] = (D)x[e];
}

template <typename T>
__global__ void k_fill(T* __restrict__ y, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    y[e] = (T)0;
}

// flag |= 1 when x holds a NaN or an infinity
template <typename T>
__global__ void k_nonfinite(const T* __restrict__ x, int64_t n, unsigned* __restrict__ flag) {
  bool bad = false;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    bad = bad || !isfinite(x[e]);
  if (bad) atomicOr(flag, 1u);
}

template <typename T>
__global__ void k_add_const(T* __restrict__ y, const double* __restrict__ cdev, int ncomp, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ncomp; e += (int64_t)gridDim.x * blockDim.x)
    y[e] = (T)((double)y[e] + cdev[e / n]);
}

template <typename T>
__global__ __launch_bounds__(256) void k_grid_partial(const T* __restrict__ x, int64_t n, int nblk,
                                                      double* __restrict__ partial) {
  __shared__ double red[256];
  const int comp = blockIdx.y;
  const T* xc = x + comp * n;
  double s = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)nblk * 256) s += (double)xc[e];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[comp * nblk + blockIdx.x] = red[0];
}

__global__ void k_partial_final(const double* __restrict__ partial, int nblk, double scale, double* __restrict__ out) {
  const int comp = blockIdx.x;
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int b = 0; b < nblk; ++b) s += partial[comp * nblk + b];
    out[comp] = s * scale;
  }
}

inline unsigned grid_blocks(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (unsigned)(b > 8192 ? 8192 : (b < 1 ? 1 : b));
}

}  // namespace

void markers_setup(const MarkerGeom& g, int kernel, int64_t n_ib, const double* X, int* s, double* f, double* wt,
                   int* tile_count, hipStream_t st, const int* pid, int nprob) {
  const int64_t ntile = (int64_t)g.ntile[0] * g.ntile[1] * g.ntile[2] * nprob;
  IBDL_HIP(hipMemsetAsync(tile_count, 0, sizeof(int) * ntile, st));
  if (n_ib > 0)
    hipLaunchKernelGGL(k_marker_setup, dim3((unsigned)((4 * n_ib + 255) / 256)), dim3(256), 0, st, g, kernel, n_ib, X,
                       s, f, wt, tile_count, pid);
  IBDL_LAUNCH_CHECK();
}

// one workgroup per busy tile: the window starts of its candidates relative to the tile's first node
__global__ __launch_bounds__(256) void k_list_offsets(MarkerGeom g, const int4* __restrict__ busy,
                                                      const int* __restrict__ list, const int* __restrict__ s,
                                                      int* __restrict__ lofs) {
  const int4 bt = busy[blockIdx.x];
  const int tl = bt.x % (g.ntile[0] * g.ntile[1] * g.ntile[2]);
  const int o0 = (tl % g.ntile[0]) * g.tile[0];
  const int o1 = ((tl / g.ntile[0]) % g.ntile[1]) * g.tile[1];
  const int o2 = (tl / (g.ntile[0] * g.ntile[1])) * g.tile[2];
  for (int i = bt.y + (int)threadIdx.x; i < bt.z; i += (int)blockDim.x) {
    const int m = list[i];
    const int d0 = (s[3 * m] - o0) & (g.n[0] - 1), d1 = (s[3 * m + 1] - o1) & (g.n[1] - 1);
    const int d2 = (s[3 * m + 2] - o2) & (g.n[2] - 1);
    lofs[i] = d0 | (d1 << 10) | (d2 << 20);
  }
}

void markers_list_offsets(const MarkerGeom& g, const int4* busy, int nbusy, const int* list, const int* s, int* lofs,
                          hipStream_t st) {
  if (g.dim != 3) throw Error(-1, "list offsets: 3-D grids only");
  if (g.n[0] > 1024 || g.n[1] > 1024 || g.n[2] > 1024) throw Error(-1, "list offsets: axes of at most 1024 nodes");
  if (nbusy <= 0) return;
  hipLaunchKernelGGL(k_list_offsets, dim3((unsigned)nbusy), dim3(256), 0, st, g, busy, list, s, lofs);
  IBDL_LAUNCH_CHECK();
}

void markers_bin(const MarkerGeom& g, int64_t n_ib, const int* s, const int* tile_count, int* tile_off,
                 int* tile_cur, int* list, int* list_tmp, int4* busy, int4* busy_tmp, int* busy_off, hipStream_t st,
                 const int* pid, int nprob, int xcd_groups) {
  const int ntile = g.ntile[0] * g.ntile[1] * g.ntile[2] * nprob;
  hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(1024), 0, st, tile_count, tile_off, busy_off, busy_tmp, tile_cur, ntile);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_busy_order, dim3((ntile + kOrder - 1) / kOrder), dim3(256), 0, st, busy_tmp, busy_off + ntile,
                     busy, xcd_groups);
  IBDL_LAUNCH_CHECK();
  if (n_ib > 0)
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((8 * n_ib + 255) / 256)), dim3(256), 0, st, g, n_ib, s, tile_off,
                       tile_cur, list_tmp, pid);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_sort_tiles, dim3(ntile), dim3(256), 0, st, tile_off, list_tmp, list);
  IBDL_LAUNCH_CHECK();
}

void exclusive_scan(const int* cnt, int* off, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, st, cnt, off, n);
  IBDL_LAUNCH_CHECK();
}

void markers_row_segments(const MarkerGeom& g, const int* tile_off, const int* rows, int64_t nact,
                          unsigned long long* seg, hipStream_t st) {
  if (nact <= 0) return;
  hipLaunchKernelGGL(k_row_segments, dim3((unsigned)((nact * seg_row_words(g) + 255) / 256)), dim3(256), 0, st, g,
                     tile_off, rows, nact, seg);
  IBDL_LAUNCH_CHECK();
}

void markers_rows(const MarkerGeom& g, int64_t n_ib, const int* s, int* lo, int* hi, int* cnt, int* off, int2* lim,
                  int* rows, const int* nbusy, const int* tile_off, unsigned long long* seg, unsigned long long* count,
                  int* host, hipStream_t st) {
  const int nplanes = g.dim == 3 ? g.n[2] : 1;
  hipLaunchKernelGGL(k_rows_init, dim3((nplanes + 255) / 256), dim3(256), 0, st, lo, hi, nplanes, g.n[1], count);
  IBDL_LAUNCH_CHECK();
  if (n_ib > 0)
    hipLaunchKernelGGL(k_rows_mark, dim3((unsigned)((n_ib + 255) / 256)), dim3(256), sizeof(int) * 2 * nplanes, st,
                       g, n_ib, s, lo, hi);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_rows_count, dim3(1), dim3(1024), 0, st, lo, hi, nplanes, cnt, off, lim, nbusy, host);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_rows_list, dim3(nplanes), dim3(256), 0, st, lo, cnt, off, nplanes, g.n[1], rows);
  IBDL_LAUNCH_CHECK();
  const int64_t nrows = (int64_t)g.n[1] * nplanes;
  hipLaunchKernelGGL(k_all_row_segments, dim3((unsigned)((nrows * seg_row_words(g) + 255) / 256)), dim3(256), 0, st, g,
                     tile_off, nrows, lim, seg, count, host + 2 + 2 * nplanes);
  IBDL_LAUNCH_CHECK();
}


template <typename T>
void grid_fill_zero(T* y, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL((k_fill<T>), dim3(grid_blocks(n)), dim3(256), 0, st, y, n);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void nonfinite_flag(const T* x, int64_t n, unsigned* flag, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_nonfinite<T>), dim3(grid_blocks(n)), dim3(256), 0, st, x, n, flag);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void spread(const SpreadArgs& a, const cplx<T>* wtab, T* out, hipStream_t st) {
  // nodes outside the non-empty tiles are not written: the caller clears the fields first
  if (a.nbusy == 0) return;
  const bool one = a.nf == 1;
  if (a.g.dim == 2) {
    if (one) hipLaunchKernelGGL((k_spread2<T, 1>), dim3(a.nbusy), dim3(256), 0, st, a, wtab, out);
    else hipLaunchKernelGGL((k_spread2<T, 5>), dim3(a.nbusy), dim3(256), 0, st, a, wtab, out);
  } else {
    if (a.mode == SP_STOKES) throw Error(-1, "3-D spread: the Stokes mode is two-dimensional");
    constexpr int NW = kSpreadWaves, SC = kSpreadCands;
    if (one && a.mode == SP_FDDIV && a.lofs)
      hipLaunchKernelGGL((k_spread3f<T, NW, SC>), dim3(a.nbusy), dim3(64 * NW), 0, st, a, wtab, out);
    else if (one && a.mode == SP_FDDIV)
      hipLaunchKernelGGL((k_spread3m<T, 1, true, NW, SC>), dim3(a.nbusy), dim3(64 * NW), 0, st, a, wtab, out);
    else if (one)
      hipLaunchKernelGGL((k_spread3m<T, 1, false, NW, SC>), dim3(a.nbusy), dim3(64 * NW), 0, st, a, wtab, out);
    else
      hipLaunchKernelGGL((k_spread3m<T, 5, false, NW, SC>), dim3(a.nbusy), dim3(64 * NW), 0, st, a, wtab, out);
  }
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void spread2_queue(const SpreadGroup* gd, const int2* items, int nitems, const double* qbase, int nblocks,
                   hipStream_t st) {
  if (nitems <= 0) return;
  const int nb = nblocks > 0 ? (nblocks < nitems ? nblocks : nitems) : nitems;
  hipLaunchKernelGGL((k_spread2_queue<T>), dim3((unsigned)nb), dim3(256), 0, st, gd, items, nitems, qbase);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void interp4_groups(const InterpGroup* gd, int ng, int64_t ntot_m, const double* xbase, double* out, hipStream_t st) {
  if (ntot_m <= 0) return;
  const int64_t lanes = ntot_m * 4;
  hipLaunchKernelGGL((k_interp4_groups<T>), dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st, gd, ng, ntot_m,
                     xbase, out);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void weight_table(const double* wt, int64_t n_ib, cplx<T>* tab, hipStream_t st) {
  const int64_t n = n_ib * 24;
  if (n > 0) hipLaunchKernelGGL((k_wtab<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, wt, n_ib, tab);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void interp(const InterpArgs& a, const cplx<T>* wtab, const T* u, double* out, hipStream_t st, const BorderArgs& bd) {
  if (a.n_ib == 0) return;
  if (a.nf < 1 || a.nf > 5) throw Error(-1, "interp: 1..5 fields");
  const bool six = a.kernel == KID_BSPLINE6;
  const int64_t lanes = six ? a.n_ib : a.n_ib * (a.g.dim == 3 ? 16 : 4);
  const int nm = (int)((lanes + 255) / 256);
  const dim3 grid((unsigned)(nm + (bd.q ? bd.nq : 0)));
  auto four = [&](auto dc, auto nc) {
    constexpr int D = decltype(dc)::value, NF = decltype(nc)::value;
    if (bd.q) hipLaunchKernelGGL((k_interp4_border<T, D, NF>), grid, dim3(256), 0, st, a, wtab, u, out, nm, bd);
    else hipLaunchKernelGGL((k_interp4<T, D, NF>), grid, dim3(256), 0, st, a, wtab, u, out);
  };
  using std::integral_constant;
  using d2 = integral_constant<int, 2>;
  using d3 = integral_constant<int, 3>;
  if (six) {
    if (a.g.dim == 2) hipLaunchKernelGGL((k_interp<T, 2, 6>), grid, dim3(256), 0, st, a, u, out, nm, bd);
    else hipLaunchKernelGGL((k_interp<T, 3, 6>), grid, dim3(256), 0, st, a, u, out, nm, bd);
  } else if (a.g.dim == 2) {
    if (a.nf == 1) four(d2{}, integral_constant<int, 1>{});
    else if (a.nf == 2) four(d2{}, integral_constant<int, 2>{});
    else four(d2{}, integral_constant<int, 5>{});
  } else {
    if (a.nf == 1) four(d3{}, integral_constant<int, 1>{});
    else four(d3{}, integral_constant<int, 5>{});
  }
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void interp_adj(const InterpArgs& a, const AdjArgs& ad, const cplx<T>* wtab, const T* u, double* y, hipStream_t st,
                const BorderArgs& bd) {
  if (a.n_ib == 0) return;
  if (a.kernel == KID_BSPLINE6 || a.nf < 1 || a.nf > 5) throw Error(-2, "interp_adj: 4-point kernels, 1..5 fields");
  const int nm = (int)((a.n_ib * (a.g.dim == 3 ? 16 : 4) + 255) / 256);
  const dim3 grid((unsigned)(nm + (bd.q ? bd.nq : 0)));
  if (a.g.dim == 2) hipLaunchKernelGGL((k_interp4_adj<T, 2>), grid, dim3(256), 0, st, a, ad, wtab, u, y, nm, bd);
  else hipLaunchKernelGGL((k_interp4_adj<T, 3>), grid, dim3(256), 0, st, a, ad, wtab, u, y, nm, bd);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void interp_div(const InterpArgs& a, const cplx<T>* wtab, const T* u, const double* nrm, const double* ds, double eta,
                double hDinv, const double* pu, double* y, hipStream_t st, const BorderArgs& bd) {
  if (a.n_ib == 0) return;
  if (a.kernel == KID_BSPLINE6) throw Error(-2, "interp_div: 4-point kernels only");
  const int64_t lanes = a.n_ib * (a.g.dim == 3 ? 32 : 8);
  const int nm = (int)((lanes + 255) / 256);
  const dim3 grid((unsigned)(nm + (bd.q ? bd.nq : 0)));
  if (a.g.dim == 2)
    hipLaunchKernelGGL((k_interp_div<T, 2>), grid, dim3(256), 0, st, a, wtab, u, nrm, ds, eta, hDinv, pu, y, nm, bd);
  else hipLaunchKernelGGL((k_interp_div<T, 3>), grid, dim3(256), 0, st, a, wtab, u, nrm, ds, eta, hDinv, pu, y, nm, bd);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void gather_dx(const GatherArgs& a, hipStream_t st) {
  if (a.n_ib == 0) return;
  if (a.nfield < 1 || a.nfield > 8) throw Error(-1, "gather_dx: 1..8 fields");
  const dim3 grid((unsigned)((a.n_ib * kGatherLanes + 255) / 256));
  const bool six = a.kernel == KID_BSPLINE6;
  if (a.g.dim == 2) {
    if (six) hipLaunchKernelGGL((k_gather_dx<T, 2, 6>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_gather_dx<T, 2, 4>), grid, dim3(256), 0, st, a);
  } else {
    if (six) hipLaunchKernelGGL((k_gather_dx<T, 3, 6>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_gather_dx<T, 3, 4>), grid, dim3(256), 0, st, a);
  }
  IBDL_LAUNCH_CHECK();
}

void grid_widen(const float* x, double* y, int64_t n, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL((k_convert<float, double>), dim3(grid_blocks(n)), dim3(256), 0, st, x, y, n);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void grid_axpby(T* y, double a, const T* x, double b, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL((k_axpby<T>), dim3(grid_blocks(n)), dim3(256), 0, st, y, a, x, b, n);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void grid_add_const(T* y, const double* c_dev, int ncomp, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL((k_add_const<T>), dim3(grid_blocks(n * ncomp)), dim3(256), 0, st, y, c_dev, ncomp, n);
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void grid_sum(const T* x, int ncomp, int64_t n, double* partial, int nblk, double* out, hipStream_t st) {
  hipLaunchKernelGGL((k_grid_partial<T>), dim3(nblk, ncomp), dim3(256), 0, st, x, n, nblk, partial);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_partial_final, dim3(ncomp), dim3(64), 0, st, partial, nblk, 1.0, out);
  IBDL_LAUNCH_CHECK();
}

#define IBDL_IB_INST(T)                                                                   \
  template void spread<T>(const SpreadArgs&, const cplx<T>*, T*, hipStream_t);            \
  template void weight_table<T>(const double*, int64_t, cplx<T>*, hipStream_t);           \
  template void grid_fill_zero<T>(T*, int64_t, hipStream_t);                              \
  template void nonfinite_flag<T>(const T*, int64_t, unsigned*, hipStream_t);             \
  template void interp<T>(const InterpArgs&, const cplx<T>*, const T*, double*, hipStream_t, const BorderArgs&); \
  template void interp_adj<T>(const InterpArgs&, const AdjArgs&, const cplx<T>*, const T*, double*, hipStream_t, \
                              const BorderArgs&);                                          \
  template void interp_div<T>(const InterpArgs&, const cplx<T>*, const T*, const double*, const double*, double, \
                              double, const double*, double*, hipStream_t, const BorderArgs&); \
  template void grid_axpby<T>(T*, double, const T*, double, int64_t, hipStream_t);        \
  template void gather_dx<T>(const GatherArgs&, hipStream_t);                             \
  template void grid_add_const<T>(T*, const double*, int, int64_t, hipStream_t);          \
  template void grid_sum<T>(const T*, int, int64_t, double*, int, double*, hipStream_t);  \
  template void spread2_queue<T>(const SpreadGroup*, const int2*, int, const double*, int, hipStream_t); \
  template void interp4_groups<T>(const InterpGroup*, int, int64_t, const double*, double*, hipStream_t);
IBDL_IB_INST(float)
IBDL_IB_INST(double)

}  // namespace ibdl
