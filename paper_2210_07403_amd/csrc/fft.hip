// FFT passes of three-dimensional grids for gfx950 (wave64), hand-written Stockham autosort
// (fft_core.h).
//
// Passes:  x axis  real <-> half spectrum, by an N/2-point complex FFT of (x_2n + i x_2n+1)
//                  and the standard even/odd split; a row belongs to one wave.
//          strided in-place C2C along y (the middle axis), tiles of W adjacent lines so each
//                  row of the tile is one contiguous segment.
//          fused   last axis: forward FFT of every input field, Fourier multiplier of the scalar
//                  operators, inverse FFT of the output fields, in one kernel: the spectra never
//                  go back to HBM.
#include "fft_core.h"
#include "kernels.h"

namespace ibdl {
namespace {

constexpr int kBlock = 256;
constexpr int kLdsBytes = 65536;
// The single-field line passes (strided, and the fused scalar pass) take up to 512 threads and
// 96 KiB of LDS per workgroup (gfx950 gives a workgroup up to 160 KiB): a tile of 32 lines of 256
// float points, 256-byte segments per row.  The multi-field passes keep 256 threads, which leaves
// their lines the registers they need.
constexpr int kLineBlock = 512;
constexpr int kLineLds = 98304;

// Global loads / stores of a line's register elements i + s*T: element o0 + (i + s*T) * es of the
// launch-uniform array base.  Addresses are base plus a 32-bit byte offset (the launchers check
// that no launch spans 4 GiB), i.e. a scalar base and one 32-bit register per access.  One
// validity branch per line; the row mask is uniform across the launch, so its test is a scalar
// branch around the masked form.
template <int N, int RMX, typename C>
__device__ __forceinline__ void line_gload(C* v, const C* __restrict__ base, unsigned o0, unsigned es, int i,
                                           bool valid, const RowMask& m) {
  constexpr int RM = RMX, TT = Plan<N, RMX>::T;
  if (!valid) {
#pragma unroll
    for (int s = 0; s < RM; ++s) v[s] = mk<C>(0, 0);
    return;
  }
  const unsigned b0 = (o0 + (unsigned)i * es) * (unsigned)sizeof(C), step = TT * es * (unsigned)sizeof(C);
  if (m.load) {
#pragma unroll
    for (int s = 0; s < RM; ++s) {
      const int y = i + s * TT;
      v[s] = (y >= m.lo && y <= m.hi) ? at(base, b0 + s * step) : mk<C>(0, 0);
    }
  } else {
#pragma unroll
    for (int s = 0; s < RM; ++s) v[s] = at(base, b0 + s * step);
  }
}

template <int N, int RMX, typename C>
__device__ __forceinline__ void line_gstore(const C* v, C* __restrict__ base, unsigned o0, unsigned es, int i,
                                            bool valid, const RowMask& m) {
  constexpr int RM = RMX, TT = Plan<N, RMX>::T;
  if (!valid) return;
  const unsigned b0 = (o0 + (unsigned)i * es) * (unsigned)sizeof(C), step = TT * es * (unsigned)sizeof(C);
  if (m.store) {
#pragma unroll
    for (int s = 0; s < RM; ++s) {
      const int y = i + s * TT;
      if (y >= m.lo && y <= m.hi) at(base, b0 + s * step) = v[s];
    }
  } else {
#pragma unroll
    for (int s = 0; s < RM; ++s) at(base, b0 + s * step) = v[s];
  }
}

// Full line transform on registers v (pattern i + s*T).  All threads of the block must call it
// (it contains block barriers when N needs more than one stage).  lds: this line's exchange
// buffer with element stride es; the caller must not rely on its contents afterwards.
template <int N, bool INV, bool BATCH = false, int RMX = plan_rmax(N), int S = 0, typename C>
__device__ __forceinline__ void fft_line(C* v, int i, C* lds, int es, const C* __restrict__ tw, int tws) {
  if constexpr (S < Plan<N, RMX>::NST) {
    stage_compute<N, S, INV, BATCH, RMX>(v, i, tw, tws);
    if constexpr (S + 1 < Plan<N, RMX>::NST) {
      __syncthreads();
      stage_store<N, S, RMX>(v, i, lds, es);
      __syncthreads();
      line_load<N, RMX>(v, i, lds, es);
    }
    fft_line<N, INV, BATCH, RMX, S + 1>(v, i, lds, es, tw, tws);
  }
}

// copy n twiddles tw[e * tws] into LDS at dst; the first read follows a block barrier
template <typename C>
__device__ __forceinline__ const C* stage_table(C* dst, const C* __restrict__ tw, int n, int tid, int nthr,
                                                int tws = 1) {
  for (int e = tid; e < n; e += nthr) dst[e] = tw[e * tws];
  return dst;
}

// ------------------------------------------------------------------ x axis
// Rows of M = nx / 2 complex points, T = M / RMX <= 64 threads each, so that a row belongs to one wave
// and its exchanges need no workgroup barrier: a thread loads its elements of the row from memory,
// transforms, takes the mirrored mode of the even/odd split through LDS and stores (or the reverse).
// Bound by HBM on a large grid (512^3 FP64, all rows: 412 and 425 us, 5.2 and 5.1 TB/s, a copy's rate)
// and by the latency of one load - transform - store chain on a row list (256^3 sphere, 10k rows, FP32:
// 9.7 and 10.5 us).  With rows staged in LDS by the whole block, the twiddles beside them and a workgroup
// barrier per exchange these were 458 / 464 and 13 / 13 us.  Eight elements per thread; single precision
// rows of 128 values and more take sixteen, two stages instead of three (512^3, all rows: 248 and 272 us
// with eight, 221 and 248 with sixteen; the 256^3 row list the same; double the same).
template <typename TR, int M> struct RowCfg {
  static constexpr int RMX = sizeof(TR) == 4 && M >= 128 ? 16 : 8;
  static constexpr int T = M / RMX;
  static constexpr int LS = pad_len(M) + 4;              // LDS row stride: an exchange line, or M + 1 modes
  static constexpr int RPB = kBlock / T;                 // most rows per block
  static_assert(T <= 64, "a row belongs to one wave");
};

// forward R2C; TI: element type of the input rows (float rows widened on load for a double transform)
template <typename T, int M, typename TI = T>
__global__ __launch_bounds__(kBlock) void k_x_r2c(const TI* __restrict__ in, cplx<T>* __restrict__ out, unsigned nrows,
                                                  const cplx<T>* __restrict__ tw, const cplx<T>* __restrict__ st,
                                                  RowList rl, int pitch) {
  using C = cplx<T>;
  using RC = RowCfg<T, M>;
  constexpr int RMX = RC::RMX, TT = RC::T;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lrow = tid / TT, i = tid - lrow * TT;
  const unsigned r = blockIdx.x * (blockDim.x / TT) + lrow;
  const bool live = r < nrows;
  const unsigned rc = live ? r : nrows - 1;
  const int64_t row = rl.row(rc);
  const unsigned long long seg = live ? rl.segmask(rc) : 0ull;
  const int64_t srow = live ? rl.sub_row(rc) : -1;
  const cplx<TI>* src = reinterpret_cast<const cplx<TI>*>(in) + row * M;
  C v[1][RMX];
#pragma unroll
  for (int s = 0; s < RMX; ++s) {
    v[0][s] = mk<C>(0, 0);
    if ((seg >> ((i + s * TT) >> rl.seg_log2)) & 1ull) {
      const cplx<TI> x = src[i + s * TT];
      v[0][s] = mk<C>((T)x.x, (T)x.y);
    }
  }
  if (srow >= 0) {   // minus a dense forcing
    const C* sub = static_cast<const C*>(rl.sub) + srow * M;
#pragma unroll
    for (int s = 0; s < RMX; ++s) v[0][s] = csub(v[0][s], sub[i + s * TT]);
  }
  C wk[RMX];
#pragma unroll
  for (int s = 0; s < RMX; ++s) wk[s] = tw[i + s * TT];
  C* line = reinterpret_cast<C*>(smem) + lrow * RC::LS;
  C w0[RMX];
  int par = 0;
  fft_multi<M, false, 1, RMX, 1>(v, i, line, 0, par, st, w0);
  line_sync<TT>();
#pragma unroll
  for (int s = 0; s < RMX; ++s) line[i + s * TT] = v[0][s];
  line_sync<TT>();
  if (!live) return;
  C* dst = out + row * pitch;
#pragma unroll
  for (int s = 0; s < RMX; ++s) {
    const int k = i + s * TT;
    const C zk = v[0][s], zm = line[k == 0 ? 0 : M - k];
    const C E = mk<C>((zk.x + zm.x) * (T)0.5, (zk.y - zm.y) * (T)0.5);
    const C O = mk<C>((zk.y + zm.y) * (T)0.5, -(zk.x - zm.x) * (T)0.5);
    dst[k] = cadd(E, cmul(wk[s], O));
    if (k == 0) dst[M] = mk<C>(zk.x - zk.y, (T)0);
  }
}

// inverse C2R
template <typename T, int M>
__global__ __launch_bounds__(kBlock) void k_x_c2r(const cplx<T>* __restrict__ in, T* __restrict__ out, unsigned nrows,
                                                  const cplx<T>* __restrict__ tw, const cplx<T>* __restrict__ st,
                                                  RowList rl, int pitch) {
  using C = cplx<T>;
  using RC = RowCfg<T, M>;
  constexpr int RMX = RC::RMX, TT = RC::T;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lrow = tid / TT, i = tid - lrow * TT;
  const unsigned r = blockIdx.x * (blockDim.x / TT) + lrow;
  const bool live = r < nrows;
  const int64_t row = rl.row(live ? r : nrows - 1);
  const C* src = in + row * pitch;
  C x[RMX], last = mk<C>(0, 0);
#pragma unroll
  for (int s = 0; s < RMX; ++s) x[s] = src[i + s * TT];
  if (i == 0) last = src[M];
  C wk[RMX];
#pragma unroll
  for (int s = 0; s < RMX; ++s) wk[s] = tw[i + s * TT];
  C* line = reinterpret_cast<C*>(smem) + lrow * RC::LS;
#pragma unroll
  for (int s = 0; s < RMX; ++s) line[i + s * TT] = x[s];
  if (i == 0) line[M] = last;
  line_sync<TT>();
  // Z'_k = (X_k + conj X_{M-k}) + i conj(W^k) (X_k - conj X_{M-k})
  C v[1][RMX];
#pragma unroll
  for (int s = 0; s < RMX; ++s) {
    const C a = x[s], b = line[M - (i + s * TT)];
    v[0][s] = cadd(mk<C>(a.x + b.x, a.y - b.y), cmul(mk<C>(wk[s].y, wk[s].x), mk<C>(a.x - b.x, a.y + b.y)));
  }
  C w0[RMX];
  int par = 0;
  fft_multi<M, true, 1, RMX, 1>(v, i, line, 0, par, st, w0);
  if (!live) return;
  C* dst = reinterpret_cast<C*>(out) + row * M;
#pragma unroll
  for (int s = 0; s < RMX; ++s) dst[i + s * TT] = v[0][s];
}

// tile width (lines per block) for strided and fused passes
// elements per thread of the strided and fused passes: at most 8 in double precision up to N = 256,
// whose 16-element lines need more registers than leave room for a second wave per SIMD (longer
// lines keep 16, or their tiles would narrow below 64-byte segments)
template <typename T> constexpr int rmax_t(int N) {
  return sizeof(T) == 8 && N <= 256 && plan_rmax(N) > 8 ? 8 : plan_rmax(N);
}
// Elements per thread of the general fused last-axis passes: the 1024-point double ones hold 8 instead
// of 16, which keeps them clear of register spills (the single-field pass k_fused1 keeps the default).
template <typename T> constexpr int fused_rmax(int N) {
  return plan_rmax(N) > 8 && sizeof(T) == 8 && N >= 1024 ? 8 : rmax_t<T>(N);
}
template <typename T, int N, int RX = rmax_t<T>(N), int BLK = kBlock, int LDS = kLdsBytes> struct TileCfg {
  static constexpr int RMX = RX;
  static constexpr int T_ = Plan<N, RMX>::T;
  static constexpr int W0 = BLK / T_;
  static constexpr int WL = LDS / (N * (int)sizeof(cplx<T>));
  // lines per tile: a power of two (the kernels split a thread index into line and element by it)
  static constexpr int W = pow2floor((W0 < WL ? W0 : WL) > 0 ? (W0 < WL ? W0 : WL) : 1);
  static constexpr int NT = W * T_;  // threads per block
  // twiddles staged in LDS when the table fits beside the widest tile (all but 1024 in double)
  static constexpr bool TWL = (W * N + N) * (int)sizeof(cplx<T>) <= LDS;
};
// the single-field passes' tile configuration
template <typename T, int N, int RX = rmax_t<T>(N)> using LineCfg = TileCfg<T, N, RX, kLineBlock, kLineLds>;
// Radix plans of the single-field line passes: plan 0 holds rmax_t elements per thread, plan 1 half
// as many (twice the threads per line, one more radix stage) where that leaves at least 4 and a line
// fits a workgroup; the launch-shape timing picks one per pass.
template <typename T> constexpr int plan_rx(int N, int plan) {
  return plan == 1 && rmax_t<T>(N) >= 8 && N / (rmax_t<T>(N) / 2) <= kLineBlock ? rmax_t<T>(N) / 2 : rmax_t<T>(N);
}

// Tile of this workgroup in the strided and last-axis passes.  A tile of W lines reads and writes
// W adjacent elements of each row; when they fill less than a 128-byte cache line the line is
// shared with the neighbouring tiles, which are then kept on one XCD so that it is fetched into one
// L2 once rather than into several.
template <typename C> __device__ __forceinline__ unsigned tile_of_block(int W) {
  return W * (int)sizeof(C) < 128 ? (unsigned)xcd_chunk((int)blockIdx.x, (int)gridDim.x) : blockIdx.x;
}

// Lines of the last-axis passes come in rows of `inner`: x modes 0 .. vinner - 1, then pitch
// padding.  With tiles of W consecutive lines, a row's last tile holds its last x mode (the Nyquist
// one) beside W - 1 padding lines: at 256 points along x, one tile in nine.  Where W divides
// vinner - 1 (both powers of two) the tiles are assigned instead as LineMap on = 1 describes, so that
// no tile holds padding; the tiles of last modes read W rows' lines (1 / (vinner - 1) of the data,
// but one cache line per element and row) and come first, so that they do not finish last.  (The
// strided passes keep the plain assignment: there the gathered last-mode tiles cost more than the
// padding lines did.)
inline LineMap line_map(int64_t nlines, int64_t inner, int64_t vinner, int W, int64_t* nblocks) {
  LineMap m;
  const int64_t lead = vinner - 1;
  const auto pow2 = [](int64_t v) { return v > 0 && (v & (v - 1)) == 0; };
  if (inner > vinner && W >= 1 && pow2(W) && lead >= W && lead % W == 0 && pow2(lead / W) && nlines % inner == 0 &&
      nlines / inner <= (int64_t)UINT32_MAX / 2) {
    m.on = 1;
    m.lw = __builtin_ctzll((unsigned long long)W);
    m.lm = __builtin_ctzll((unsigned long long)(lead / W));
    m.rows = (unsigned)(nlines / inner);
    m.nlast = (unsigned)(((int64_t)m.rows + W - 1) / W);
    *nblocks = (int64_t)m.nlast + (int64_t)m.rows * (lead / W);
  } else {
    *nblocks = (nlines + W - 1) / W;
  }
  return m;
}

// row lq and x mode li of column c of tile t; false for padding and for lines past the last row
__device__ __forceinline__ bool tile_lines(const LineMap& m, unsigned t, int c, int W, unsigned inner,
                                           unsigned vinner, int64_t nlines, unsigned& lq, unsigned& li) {
  if (m.on) {
    if (t < m.nlast) {   // last x modes: strided rows, slower per tile, so dispatched first
      lq = (t << m.lw) + (unsigned)c;
      li = vinner - 1;
      return lq < m.rows;
    }
    t -= m.nlast;
    lq = t >> m.lm;
    li = ((t & ((1u << m.lm) - 1u)) << m.lw) + (unsigned)c;
    return true;
  }
  const unsigned l = t * (unsigned)W + (unsigned)c;
  lq = l / inner;
  li = l - lq * inner;
  return l < nlines && li < vinner;
}

// ------------------------------------------------------------------ strided in-place C2C
template <typename T, int N, bool INV, int RX = rmax_t<T>(N)>
__global__ __launch_bounds__(kLineBlock) void k_strided(cplx<T>* __restrict__ data, int64_t nlines, int64_t inner,
                                                        int64_t outer, int64_t es, const cplx<T>* __restrict__ twg,
                                                        int W, RowMask rm, int64_t vinner) {
  using C = cplx<T>;
  using TC = LineCfg<T, N, RX>;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  const int tid = threadIdx.x;
  const C* tw = TC::TWL ? stage_table(lds + N * W, twg, N, tid, W * TC::T_) : twg;
  const int c = tid & (W - 1), i = tid / W;
  const unsigned l = tile_of_block<C>(W) * (unsigned)W + c;
  const unsigned lq = l / (unsigned)inner, li = l - lq * (unsigned)inner;
  const bool valid = l < nlines && li < vinner;
  const unsigned lp = rm.phys_plane(lq);
  const unsigned base = valid ? lp * (unsigned)outer + li : 0u;
  const RowMask pm = rm.plane(valid ? lp : 0);   // rows of this line's plane that matter
  C v[TC::RMX];
  line_gload<N, TC::RMX>(v, data, base, (unsigned)es, i, valid, pm);
  fft_line<N, INV, !TC::TWL, TC::RMX>(v, i, lds + c, W, tw, 1);
  line_gstore<N, TC::RMX>(v, data, base, (unsigned)es, i, valid, pm);
}

// ------------------------------------------------------------------ Fourier multiplier
// u^ = alpha*sc * (sum_f c_f F^_f) / (c2*sigma - c0), c_f = i k~_d (FK_D*) or 1 (FK_MASS); zero where
// c2*sigma - c0 = 0 (mean-zero inverse).
// Line l = jy nxp + jx of the (jy, jx) plane, elements strided by the plane size P; element e is mode e.
template <typename T, int N>
__global__ __launch_bounds__(kBlock) void k_fused(cplx<T>* __restrict__ data, int64_t P, MultDesc md,
                                                  const cplx<T>* __restrict__ twg, int W, int64_t bstride, RowMask rm) {
  using C = cplx<T>;
  using TC = TileCfg<T, N, fused_rmax<T>(N)>;
  constexpr int RM = TC::RMX, TT = TC::T_;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  data += (int64_t)blockIdx.y * bstride;   // problem of a batch
  const int tid = threadIdx.x;
  const C* tw = TC::TWL ? stage_table(lds + N * W, twg, N, tid, W * TC::T_) : twg;
  const int c = tid & (W - 1), i = tid / W;
  unsigned lq_, li_;   // row and x mode of this thread's line; padding lines are skipped
  const bool valid = tile_lines(md.map, tile_of_block<C>(W), c, W, (unsigned)md.nxp, (unsigned)md.nxh, P, lq_, li_);
  const unsigned l = lq_ * (unsigned)md.nxp + li_;
  const int64_t FS = P * N;
  const int jx = (int)(valid ? li_ : 0u);
  const int jy = (int)(valid ? lq_ : 0u);
  const T* sgl = static_cast<const T*>(md.sig[2]);   // symbols along the line
  const T* ktl_ = static_cast<const T*>(md.kt[2]);
  const T sig_l = static_cast<const T*>(md.sig[0])[jx] + static_cast<const T*>(md.sig[1])[jy];
  const T ktl[2] = {static_cast<const T*>(md.kt[0])[jx], static_cast<const T*>(md.kt[1])[jy]};
  C acc[RM];
  T gfac[RM];   // multiplier alpha*sc / (c2 sigma - c0)
#pragma unroll
  for (int s = 0; s < RM; ++s) {
    acc[s] = mk<C>(0, 0);
    const T den = (T)md.c2 * (sig_l + sgl[i + s * TT]) - (T)md.c0;
    gfac[s] = den == (T)0 ? (T)0 : (T)(md.alpha * md.sc) * recip(den);
  }
  for (int f = 0; f < md.nc; ++f) {
    C v[RM];
    line_gload<N, RM>(v, data, (unsigned)(f * FS + l), (unsigned)P, i, valid, rm);
    fft_line<N, false, !TC::TWL, RM>(v, i, lds + c, W, tw, 1);
    const int fk = md.fk[f];
    if (fk == FK_MASS) {
#pragma unroll
      for (int s = 0; s < RM; ++s) acc[s] = cadd(acc[s], cscale(v[s], gfac[s]));
    } else if (fk == FK_DZ) {   // derivative along the line axis: k~ varies per element
#pragma unroll
      for (int s = 0; s < RM; ++s) acc[s] = cadd(acc[s], mul_ir(v[s], gfac[s] * ktl_[i + s * TT]));
    } else {                 // derivative across lines: k~ is constant on the line
      const T kc = ktl[fk];
#pragma unroll
      for (int s = 0; s < RM; ++s) acc[s] = cadd(acc[s], mul_ir(v[s], gfac[s] * kc));
    }
  }
  fft_line<N, true, !TC::TWL, RM>(acc, i, lds + c, W, tw, 1);
  line_gstore<N, RM>(acc, data, l, (unsigned)P, i, valid, rm);
}

// Single scalar field (the finite-difference operator and the scalar grid solve): forward FFT,
// multiply by the real factor alpha*sc / (c2 sigma - c0) in registers, inverse FFT.
template <typename T, int N, int RX = rmax_t<T>(N)>
__global__ __launch_bounds__(kLineBlock) void k_fused1(cplx<T>* __restrict__ data, int64_t P, MultDesc md,
                                                       const cplx<T>* __restrict__ twg, int W, int64_t bstride,
                                                       RowMask rm) {
  using C = cplx<T>;
  using TC = LineCfg<T, N, RX>;   // one field, one real factor: no spills at 16 elements per thread
  constexpr int RM = TC::RMX, TT = TC::T_;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  data += (int64_t)blockIdx.y * bstride;   // problem of a batch
  const int tid = threadIdx.x;
  const C* tw = TC::TWL ? stage_table(lds + N * W, twg, N, tid, W * TC::T_) : twg;
  const int c = tid & (W - 1), i = tid / W;
  unsigned lq_, li_;   // row and x mode of this thread's line; padding lines are skipped
  const bool valid = tile_lines(md.map, tile_of_block<C>(W), c, W, (unsigned)md.nxp, (unsigned)md.nxh, P, lq_, li_);
  const unsigned l = lq_ * (unsigned)md.nxp + li_;
  const int jx = (int)(valid ? li_ : 0u);
  const int jy = (int)(valid ? lq_ : 0u);
  const T* sgl = static_cast<const T*>(md.sig[2]);
  const T sig_l = static_cast<const T*>(md.sig[0])[jx] + static_cast<const T*>(md.sig[1])[jy];
  C v[RM];
  line_gload<N, RM>(v, data, l, (unsigned)P, i, valid, rm);
  fft_line<N, false, !TC::TWL, RM>(v, i, lds + c, W, tw, 1);
  const T num = (T)(md.alpha * md.sc), c2 = (T)md.c2, c0 = (T)md.c0;
#pragma unroll
  for (int s = 0; s < RM; ++s) {
    const T den = c2 * (sig_l + sgl[i + s * TT]) - c0;
    v[s] = cscale(v[s], den == (T)0 ? (T)0 : num * recip(den));
  }
  fft_line<N, true, !TC::TWL, RM>(v, i, lds + c, W, tw, 1);
  line_gstore<N, RM>(v, data, l, (unsigned)P, i, valid, rm);
}

// Gradient outputs (mode 1): the input spectrum stays in registers after its forward FFT and the no
// outputs i k~_o g F^ (o < 3), g F^ are formed, inverse transformed and stored one at a time (the
// input is read before the first store, and each workgroup owns its lines in every field).
template <typename T, int N>
__global__ __launch_bounds__(kBlock) void k_fused_grad(cplx<T>* __restrict__ data, int64_t P, int no, MultDesc md,
                                                       const cplx<T>* __restrict__ twg, int W, int64_t bstride,
                                                       RowMask rm) {
  using C = cplx<T>;
  using TC = TileCfg<T, N, fused_rmax<T>(N)>;
  constexpr int RM = TC::RMX, TT = TC::T_;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  data += (int64_t)blockIdx.y * bstride;   // problem of a batch
  const int tid = threadIdx.x;
  const C* tw = TC::TWL ? stage_table(lds + N * W, twg, N, tid, W * TC::T_) : twg;
  const int c = tid & (W - 1), i = tid / W;
  unsigned lq_, li_;   // row and x mode of this thread's line; padding lines are skipped
  const bool valid = tile_lines(md.map, tile_of_block<C>(W), c, W, (unsigned)md.nxp, (unsigned)md.nxh, P, lq_, li_);
  const unsigned l = lq_ * (unsigned)md.nxp + li_;
  const int64_t FS = P * N;
  const int jx = (int)(valid ? li_ : 0u);
  const int jy = (int)(valid ? lq_ : 0u);
  const T* sgl = static_cast<const T*>(md.sig[2]);
  const T* ktl_ = static_cast<const T*>(md.kt[2]);
  const T sig_l = static_cast<const T*>(md.sig[0])[jx] + static_cast<const T*>(md.sig[1])[jy];
  const T k0 = static_cast<const T*>(md.kt[0])[jx], k1 = static_cast<const T*>(md.kt[1])[jy];
  C v[RM];
  line_gload<N, RM>(v, data, l, (unsigned)P, i, valid, rm);
  fft_line<N, false, !TC::TWL, RM>(v, i, lds + c, W, tw, 1);
  for (int o = 0; o < no; ++o) {
    C acc[RM];
#pragma unroll
    for (int s = 0; s < RM; ++s) {
      const int e = i + s * TT;
      const T den = (T)md.c2 * (sig_l + sgl[e]) - (T)md.c0;
      const T g = den == (T)0 ? (T)0 : (T)(md.alpha * md.sc) * recip(den);
      const T ko = o == 0 ? k0 : (o == 1 ? k1 : ktl_[e]);
      acc[s] = o < 3 ? mul_ir(v[s], g * ko) : cscale(v[s], g);
    }
    fft_line<N, true, !TC::TWL, RM>(acc, i, lds + c, W, tw, 1);
    line_gstore<N, RM>(acc, data, (unsigned)(o * FS + l), (unsigned)P, i, valid, rm);
  }
}

// ------------------------------------------------------------------ dispatch helpers
template <typename F> void dispatch_n(int n, F&& f) {
  switch (n) {
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    case 256: f(std::integral_constant<int, 256>{}); break;
    case 512: f(std::integral_constant<int, 512>{}); break;
    case 1024: f(std::integral_constant<int, 1024>{}); break;
    default: throw Error(-2, "unsupported FFT length " + std::to_string(n));
  }
}

// the x passes' complex length, nx / 2
template <typename F> void dispatch_m(int m, F&& f) {
  if (m == 1024) throw Error(-2, "unsupported FFT length " + std::to_string(2 * m));
  dispatch_n(m, [&](auto Mc) {
    if constexpr (decltype(Mc)::value < 1024) f(Mc);
  });
}
}  // namespace

template <typename T>
int fft_x_rpb_max(int nx) {
  int r = 0;
  dispatch_m(nx / 2, [&](auto Mc) { r = RowCfg<T, decltype(Mc)::value>::RPB; });
  return r;
}

template <typename T> size_t fft_x_table_len(int nx) {
  int r = 0;
  dispatch_m(nx / 2, [&](auto Mc) { r = stage_len<decltype(Mc)::value, RowCfg<T, decltype(Mc)::value>::RMX>(); });
  return (size_t)r + 1;
}

template <typename T> TwX<T> fft_x_table(int nx, const cplx<T>* twx, cplx<T>* dst, hipStream_t s) {
  dispatch_m(nx / 2, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value, RMX = RowCfg<T, M>::RMX;
    const int len = stage_len<M, RMX>();
    if (len > 0) hipLaunchKernelGGL((k_stages<M, RMX, cplx<T>>), dim3((len + 255) / 256), dim3(256), 0, s, dst, twx, 2);
  });
  IBDL_LAUNCH_CHECK();
  TwX<T> t;
  t.base = twx;
  t.x = dst;
  return t;
}

template <typename T>
int fft_line_w_max(int n, int plan) {
  int r = 0;
  dispatch_n(n, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    r = plan == 1 ? LineCfg<T, N, plan_rx<T>(N, 1)>::W : LineCfg<T, N>::W;
  });
  return r;
}

template <typename T>
int fft_line_plans(int n) {
  int r = 1;
  dispatch_n(n, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    r = plan_rx<T>(N, 1) != plan_rx<T>(N, 0) ? 2 : 1;
  });
  return r;
}

namespace {
int pick(int want, int max) {
  if (want <= 0 || want > max) return max;
  int v = 1;
  while (2 * v <= want) v *= 2;
  return v;
}
}  // namespace

namespace {
template <typename T, typename TI>
void x_r2c_launch(const TI* in, cplx<T>* out, int nx, int64_t nrows, const TwX<T>& tw, hipStream_t s, int rpb,
                  const RowList& rl, int64_t pitch) {
  if (nrows <= 0) return;
  if (nrows > INT32_MAX) throw Error(-2, "x FFT pass: too many rows");
  dispatch_m(nx / 2, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value;
    using RC = RowCfg<T, M>;
    const int R = pick(rpb, RC::RPB);
    hipLaunchKernelGGL((k_x_r2c<T, M, TI>), dim3((unsigned)((nrows + R - 1) / R)), dim3(R * RC::T),
                       sizeof(cplx<T>) * R * RC::LS, s, in, out, (unsigned)nrows, tw.base, tw.x, rl, (int)pitch);
  });
  IBDL_LAUNCH_CHECK();
}
}  // namespace

template <typename T>
void fft_x_r2c(const T* in, cplx<T>* out, int nx, int64_t nrows, const TwX<T>& tw, hipStream_t s, int rpb,
               const RowList& rl, int64_t pitch) {
  x_r2c_launch<T, T>(in, out, nx, nrows, tw, s, rpb, rl, pitch);
}

void fft_x_r2c_widen(const float* in, cplx<double>* out, int nx, int64_t nrows, const TwX<double>& tw, hipStream_t s, int rpb,
                     const RowList& rl, int64_t pitch) {
  x_r2c_launch<double, float>(in, out, nx, nrows, tw, s, rpb, rl, pitch);
}

template <typename T>
void fft_x_c2r(const cplx<T>* in, T* out, int nx, int64_t nrows, const TwX<T>& tw, hipStream_t s, int rpb,
               const RowList& rl, int64_t pitch) {
  if (nrows <= 0) return;
  if (nrows > INT32_MAX) throw Error(-2, "x FFT pass: too many rows");
  dispatch_m(nx / 2, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value;
    using RC = RowCfg<T, M>;
    const int R = pick(rpb, RC::RPB);
    hipLaunchKernelGGL((k_x_c2r<T, M>), dim3((unsigned)((nrows + R - 1) / R)), dim3(R * RC::T),
                       sizeof(cplx<T>) * R * RC::LS, s, in, out, (unsigned)nrows, tw.base, tw.x, rl, (int)pitch);
  });
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void fft_strided(cplx<T>* data, int n, int64_t nlines, int64_t inner, int64_t outer, int64_t es, bool inverse,
                 const cplx<T>* tw, hipStream_t s, int w, const RowMask& rm, int64_t vinner, int plan) {
  if (vinner <= 0) vinner = inner;
  if (nlines <= 0) return;
  int64_t lastp = (nlines - 1) / inner;   // last plane touched
  if (rm.pspan > 0) lastp = (lastp / rm.pspan) * rm.nplanes + rm.p0 + rm.pspan - 1;
  const int64_t span = lastp * outer + (inner - 1) + (int64_t)(n - 1) * es + 1;
  if (span * (int64_t)sizeof(cplx<T>) > (int64_t)UINT32_MAX || nlines > INT32_MAX)
    throw Error(-2, "strided FFT pass: one launch may not span 4 GiB");
  dispatch_n(n, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    auto launch = [&](auto rxc) {
      constexpr int RX = decltype(rxc)::value;
      using TC = LineCfg<T, N, RX>;
      const int W = pick(w, TC::W);
      const int64_t nb = (nlines + W - 1) / W;
      const size_t lds = sizeof(cplx<T>) * (N * W + (TC::TWL ? N : 0));
      const dim3 blk(W * TC::T_);
      if (inverse)
        hipLaunchKernelGGL((k_strided<T, N, true, RX>), dim3((unsigned)nb), blk, lds, s, data, nlines, inner, outer,
                           es, tw, W, rm, vinner);
      else
        hipLaunchKernelGGL((k_strided<T, N, false, RX>), dim3((unsigned)nb), blk, lds, s, data, nlines, inner, outer,
                           es, tw, W, rm, vinner);
    };
    if (plan == 1 && plan_rx<T>(N, 1) != plan_rx<T>(N, 0))
      launch(std::integral_constant<int, plan_rx<T>(N, 1)>{});
    else
      launch(std::integral_constant<int, plan_rx<T>(N, 0)>{});
  });
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void fft_fused_last(cplx<T>* data, int n, int64_t P, int no, const MultDesc& md, const cplx<T>* tw, hipStream_t s,
                    int batch, int64_t bstride, int w, const RowMask& rm, int plan) {
  if (batch < 1) return;
  const int64_t nf = std::max<int64_t>(std::max(md.nc, no), 1);
  if (nf * P * n * (int64_t)sizeof(cplx<T>) > (int64_t)UINT32_MAX || P > INT32_MAX)
    throw Error(-2, "fused FFT pass: one problem's fields may not span 4 GiB");
  dispatch_n(n, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    // launch shape of a kernel whose tile configuration is TC: lines per block, grid, LDS
    MultDesc mdl = md;   // with the tile map of the chosen width
    auto tiles = [&](int W) {
      int64_t nb = 0;
      mdl.map = line_map(P, md.nxp, md.nxh, W, &nb);
      return dim3((unsigned)nb, (unsigned)batch);
    };
    auto shape = [&](auto tc, int& W, dim3& grid, dim3& blk, size_t& lds) {
      using TC = decltype(tc);
      W = pick(w, TC::W);
      grid = tiles(W);
      blk = dim3(W * TC::T_);
      lds = sizeof(cplx<T>) * (N * W + (TC::TWL ? N : 0));
    };
    int W = 0;
    dim3 grid, blk;
    size_t lds = 0;
    const MultDesc& md = mdl;
    if (md.mode == 1 && md.nc == 1 && no >= 1 && no <= 4) {
      shape(TileCfg<T, N, fused_rmax<T>(N)>{}, W, grid, blk, lds);
      hipLaunchKernelGGL((k_fused_grad<T, N>), grid, blk, lds, s, data, P, no, md, tw, W, bstride, rm);
    } else if (md.mode != 0 || md.stokes || no != 1) {
      throw Error(-2, "fused pass: unsupported multiplier / output count");
    } else if (md.nc == 1 && md.fk[0] == FK_MASS) {
      if (plan == 1 && plan_rx<T>(N, 1) != plan_rx<T>(N, 0)) {
        constexpr int RX = plan_rx<T>(N, 1);
        shape(LineCfg<T, N, RX>{}, W, grid, blk, lds);
        hipLaunchKernelGGL((k_fused1<T, N, RX>), grid, blk, lds, s, data, P, md, tw, W, bstride, rm);
      } else {
        shape(LineCfg<T, N>{}, W, grid, blk, lds);
        hipLaunchKernelGGL((k_fused1<T, N>), grid, blk, lds, s, data, P, md, tw, W, bstride, rm);
      }
    } else {
      shape(TileCfg<T, N, fused_rmax<T>(N)>{}, W, grid, blk, lds);
      hipLaunchKernelGGL((k_fused<T, N>), grid, blk, lds, s, data, P, md, tw, W, bstride, rm);
    }
  });
  IBDL_LAUNCH_CHECK();
}

#define IBDL_FFT_INST(T)                                                                                   \
  template void fft_x_r2c<T>(const T*, cplx<T>*, int, int64_t, const TwX<T>&, hipStream_t, int,          \
                             const RowList&, int64_t);                                                     \
  template void fft_x_c2r<T>(const cplx<T>*, T*, int, int64_t, const TwX<T>&, hipStream_t, int,          \
                             const RowList&, int64_t);                                                     \
  template size_t fft_x_table_len<T>(int);                                                                 \
  template TwX<T> fft_x_table<T>(int, const cplx<T>*, cplx<T>*, hipStream_t);                              \
  template void fft_strided<T>(cplx<T>*, int, int64_t, int64_t, int64_t, int64_t, bool, const cplx<T>*,   \
                               hipStream_t, int, const RowMask&, int64_t, int);                            \
  template void fft_fused_last<T>(cplx<T>*, int, int64_t, int, const MultDesc&, const cplx<T>*, hipStream_t, \
                                  int, int64_t, int, const RowMask&, int);                                 \
  template int fft_x_rpb_max<T>(int);                                                                      \
  template int fft_line_w_max<T>(int, int);                                                                \
  template int fft_line_plans<T>(int);
IBDL_FFT_INST(float)
IBDL_FFT_INST(double)

}  // namespace ibdl
