// Building blocks of the FFT passes (fft.hip: 3-D, fft2d.hip: 2-D): Stockham plans, in-register
// DFTs, radix stages and their LDS exchanges.
//
// A line of N points is owned by T = N / RMAX threads; thread i holds elements i + s*T (s < RMAX) in
// registers.  Each radix-R stage does R-point DFTs in registers; stages exchange through LDS; the
// first stage reads the line in the pattern i + s*T and the last stage leaves the natural-order
// result in it, so a forward and an inverse transform chain without an LDS round trip.
#pragma once

#include "common.h"

namespace ibdl {
namespace {

constexpr int pow2floor(int v) { return v >= 2 ? 2 * pow2floor(v / 2) : 1; }

// Stockham plan of a length-N line: RMAX elements per thread (the radix of every stage but the last),
// T = N / RMAX threads per line
constexpr int plan_rmax(int N) { return (N <= 16) ? N : ((N == 32 || N == 64 || N == 512) ? 8 : 16); }
template <int N, int RMX = plan_rmax(N)> struct Plan {
  static constexpr int RMAX = RMX;
  static constexpr int T = N / RMAX;
  static constexpr int LR = ilog2c(RMAX);
  static constexpr int NFULL = ilog2c(N) / LR;
  static constexpr int REM = N >> (NFULL * LR);
  static constexpr int NST = NFULL + (REM > 1 ? 1 : 0);
  static constexpr int radix(int s) { return s < NFULL ? RMAX : REM; }
  static constexpr int pw(int s) { return 1 << (s * LR); }
};

__host__ __device__ constexpr double c16(int m) {
  return m == 0 ? 1.0 : m == 1 ? 0.92387953251128675613 : m == 2 ? 0.70710678118654752440
       : m == 3 ? 0.38268343236508977173 : m == 4 ? 0.0 : m == 5 ? -0.38268343236508977173
       : m == 6 ? -0.70710678118654752440 : -0.92387953251128675613;
}
__host__ __device__ constexpr double s16(int m) {
  return m == 0 ? 0.0 : m == 1 ? 0.38268343236508977173 : m == 2 ? 0.70710678118654752440
       : m == 3 ? 0.92387953251128675613 : m == 4 ? 1.0 : m == 5 ? 0.92387953251128675613
       : m == 6 ? 0.70710678118654752440 : 0.38268343236508977173;
}

// In-register DFT of size R (2, 4, 8, 16), natural order in and out.
template <int R, bool INV, typename C>
__device__ __forceinline__ void dft(C* x) {
  using T = decltype(C::x);
  if constexpr (R == 2) {
    C a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
  } else if constexpr (R == 4) {
    C s02 = cadd(x[0], x[2]), d02 = csub(x[0], x[2]);
    C s13 = cadd(x[1], x[3]), d13 = mul_mi<INV>(csub(x[1], x[3]));
    x[0] = cadd(s02, s13);
    x[2] = csub(s02, s13);
    x[1] = cadd(d02, d13);
    x[3] = csub(d02, d13);
  } else {
    constexpr int H = R / 2;
    C e[H], o[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
      e[j] = x[2 * j];
      o[j] = x[2 * j + 1];
    }
    dft<H, INV>(e);
    dft<H, INV>(o);
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const int m = k * (16 / R);
      C t;
      if (k == 0) {
        t = o[k];
      } else if (4 * k == R) {
        t = mul_mi<INV>(o[k]);
      } else {
        C w = mk<C>((T)c16(m), (T)(INV ? s16(m) : -s16(m)));
        t = cmul(o[k], w);
      }
      x[k] = cadd(e[k], t);
      x[k + H] = csub(e[k], t);
    }
  }
}

// BATCH (a table in global memory): all twiddles of the stage are loaded before the first is used,
// so that their loads are in flight together rather than one latency each; a table staged in LDS
// is read as it is used.
template <int N, int S, bool INV, bool BATCH, int RMX, typename C>
__device__ __forceinline__ void stage_compute(C* v, int i, const C* __restrict__ tw, int tws) {
  using P = Plan<N, RMX>;
  constexpr int R = P::radix(S), PP = P::pw(S), NB = P::RMAX / R, TT = P::T;
  if constexpr (PP > 1) {
    C w[NB][R];
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      const int k = (i + m * TT) & (PP - 1);
#pragma unroll
      for (int j = 1; j < R; ++j) w[m][j] = tw[(j * k * (N / (PP * R))) * tws];
    }
    if constexpr (BATCH) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
      for (int j = 1; j < R; ++j) {
        if (INV) w[m][j].y = -w[m][j].y;
        v[m + j * NB] = cmul(v[m + j * NB], w[m][j]);
      }
  }
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    C x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) x[j] = v[m + j * NB];
    dft<R, INV>(x);
#pragma unroll
    for (int j = 0; j < R; ++j) v[m + j * NB] = x[j];
  }
}

// exchange of a line whose elements lie es apart in LDS
template <int N, int S, int RMX, typename C>
__device__ __forceinline__ void stage_store(const C* v, int i, C* lds, int es) {
  using P = Plan<N, RMX>;
  constexpr int R = P::radix(S), PP = P::pw(S), NB = P::RMAX / R, TT = P::T;
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    const int b = i + m * TT;
    const int k = b & (PP - 1);
#pragma unroll
    for (int j = 0; j < R; ++j) lds[((b - k) * R + k + j * PP) * es] = v[m + j * NB];
  }
}

template <int N, int RMX, typename C>
__device__ __forceinline__ void line_load(C* v, int i, const C* lds, int es) {
#pragma unroll
  for (int s = 0; s < RMX; ++s) v[s] = lds[(i + s * Plan<N, RMX>::T) * es];
}

// element at a byte offset from a launch-uniform base: a scalar base and one 32-bit register per access
template <typename C> __device__ __forceinline__ const C& at(const C* base, unsigned byte) {
  return *reinterpret_cast<const C*>(reinterpret_cast<const char*>(base) + (size_t)byte);
}
template <typename C> __device__ __forceinline__ C& at(C* base, unsigned byte) {
  return *reinterpret_cast<C*>(reinterpret_cast<char*>(base) + (size_t)byte);
}

// 1/x: the hardware reciprocal in single precision (about one ulp, well inside what the float
// path resolves), an exact division in double
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }


// order a line's LDS accesses across its T threads
template <int T> __device__ __forceinline__ void line_sync() {
  if constexpr (T <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Twiddles are read from a table in stage order: stage S >= 1 of a transform holds w_N^(j k N / (PP R))
// at stage_off + (j - 1) PP + k (1 <= j < R, k < PP), so that the lanes of a wave read consecutive
// values; from the plain table w_N^m they would read N / (PP R) j values apart, a cache line per lane.
template <int N, int RMX> constexpr int stage_off(int S) {
  using P = Plan<N, RMX>;
  int o = 0;
  for (int q = 1; q < S; ++q) o += (P::radix(q) - 1) * P::pw(q);
  return o;
}
template <int N, int RMX> constexpr int stage_len() { return stage_off<N, RMX>(Plan<N, RMX>::NST); }

// the twiddles of stage S on this thread's elements: w[m * R + j] multiplies element m + j * NB
template <int N, int S, int RMX, typename C>
__device__ __forceinline__ void stage_twiddles(C (&w)[RMX], int i, const C* __restrict__ tab) {
  using P = Plan<N, RMX>;
  constexpr int R = P::radix(S), PP = P::pw(S), NB = RMX / R, TT = P::T, OFF = stage_off<N, RMX>(S);
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    const int k = (i + m * TT) & (PP - 1);
#pragma unroll
    for (int j = 1; j < R; ++j) w[m * R + j] = tab[OFF + (j - 1) * PP + k];
  }
}

// fills the stage-ordered table of an N-point transform from the plain one (w_N^m at tw[m * stride])
template <int N, int RMX, typename C> __device__ void fill_stages(C* tab, const C* tw, int stride) {
  using P = Plan<N, RMX>;
  const int t0 = (int)(blockIdx.x * blockDim.x + threadIdx.x), nt = (int)(gridDim.x * blockDim.x);
  for (int S = 1; S < P::NST; ++S) {
    const int R = P::radix(S), PP = P::pw(S), off = stage_off<N, RMX>(S);
    for (int e = t0; e < (R - 1) * PP; e += nt) {
      const int j = 1 + e / PP, k = e - (j - 1) * PP;
      tab[off + e] = tw[(int64_t)(j * k * (N / (PP * R))) * stride];
    }
  }
}
template <int N, int RMX, typename C> __global__ void k_stages(C* tab, const C* tw, int stride) {
  fill_stages<N, RMX, C>(tab, tw, stride);
}

template <int N, int S, bool INV, int RMX, typename C>
__device__ __forceinline__ void stage_dft(C (&v)[RMX], const C (&w)[RMX]) {
  using P = Plan<N, RMX>;
  constexpr int R = P::radix(S), NB = RMX / R;
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    C x[R];
    x[0] = v[m];
#pragma unroll
    for (int j = 1; j < R; ++j) {
      if constexpr (S > 0) x[j] = cmul(v[m + j * NB], INV ? cconj(w[m * R + j]) : w[m * R + j]);
      else x[j] = v[m + j * NB];
    }
    dft<R, INV>(x);
#pragma unroll
    for (int j = 0; j < R; ++j) v[m + j * NB] = x[j];
  }
}

constexpr int kPad = 3;   // one pad slot every 8 values of an exchange line
constexpr int pad_len(int n) { return n + (n >> kPad); }

// Exchange of stage S through a padded line: element e lives at pad_at(e) = e + e / 8.  Every address is
// one base per stage plus a constant: (base + offset) / 8 = base / 8 + offset / 8 for the bases and
// offsets that occur (a store's base is k < PP above a multiple of PP R, a load's i < T, and PP, T are
// powers of two), which the compiler does not see by itself: it would keep an address register per
// element and stage.
__device__ __forceinline__ int pad_at(int e) { return e + (e >> kPad); }
template <int N, int S, int RMX, typename C>
__device__ __forceinline__ void put_stage(const C (&v)[RMX], int i, C* line) {
  using P = Plan<N, RMX>;
  constexpr int R = P::radix(S), PP = P::pw(S);
  static_assert(R == RMX, "a stage that exchanges uses the full radix");
  const int k = i & (PP - 1);
  C* b = line + pad_at((i - k) * R + k);
#pragma unroll
  for (int j = 0; j < R; ++j) b[pad_len(j * PP)] = v[j];
}
template <int N, int RMX, typename C>
__device__ __forceinline__ void get_line(C (&v)[RMX], int i, const C* line) {
  const C* b = line + pad_at(i);
#pragma unroll
  for (int s = 0; s < RMX; ++s) v[s] = b[pad_len(s * Plan<N, RMX>::T)];
}

// Transforms of NF lines together (same line index of NF fields): stage by stage, each field in turn
// exchanging through one of NBUF buffers of the line (bstr apart; par: the one to use next), so that
// a field's LDS reads are in flight while the next one computes.  Each stage's twiddles serve every
// field and are loaded a stage ahead.  All threads of the block call it.
// LEAN: twiddles read when a stage begins, and the fields' work kept apart, for blocks whose threads
// have few registers.
template <int N, bool INV, int NF, int RMX, int NBUF, bool LEAN = false, int S = 0, typename C>
__device__ __forceinline__ void fft_multi(C (&v)[NF][RMX], int i, C* lds, int bstr, int& par,
                                          const C* __restrict__ tw, C (&w)[RMX]) {
  using P = Plan<N, RMX>;
  if constexpr (S < P::NST) {
    C wn[RMX];
    // (the scheduler would otherwise collect the loads of all stages at the top, for a register each)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (LEAN && S > 0) stage_twiddles<N, S, RMX>(w, i, tw);
    if constexpr (!LEAN && S + 1 < P::NST) stage_twiddles<N, S + 1, RMX>(wn, i, tw);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      if constexpr (LEAN) __builtin_amdgcn_sched_barrier(0);
      stage_dft<N, S, INV, RMX>(v[f], w);
      if constexpr (S + 1 < P::NST) {
        C* b = NBUF == 2 ? lds + par * bstr : lds;
        if constexpr (NBUF == 1) line_sync<P::T>();
        put_stage<N, S, RMX>(v[f], i, b);
        line_sync<P::T>();
        get_line<N, RMX>(v[f], i, b);
        par ^= 1;
      }
    }
    fft_multi<N, INV, NF, RMX, NBUF, LEAN, S + 1>(v, i, lds, bstr, par, tw, wn);
  }
}

}  // namespace
}  // namespace ibdl
