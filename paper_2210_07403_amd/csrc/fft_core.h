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

// LDS slot of line element e: e * es, or, for a contiguous line (es = 1) with PAD > 0, e plus one
// pad slot every 2^PAD elements, so that a stage's strided stores do not fall into the same banks
template <int PAD> __device__ __forceinline__ int lslot(int e, int es) { return PAD ? e + (e >> PAD) : e * es; }

template <int N, int S, int RMX, int PAD = 0, typename C>
__device__ __forceinline__ void stage_store(const C* v, int i, C* lds, int es) {
  using P = Plan<N, RMX>;
  constexpr int R = P::radix(S), PP = P::pw(S), NB = P::RMAX / R, TT = P::T;
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    const int b = i + m * TT;
    const int k = b & (PP - 1);
#pragma unroll
    for (int j = 0; j < R; ++j) lds[lslot<PAD>((b - k) * R + k + j * PP, es)] = v[m + j * NB];
  }
}

template <int N, int RMX, int PAD = 0, typename C>
__device__ __forceinline__ void line_load(C* v, int i, const C* lds, int es) {
#pragma unroll
  for (int s = 0; s < RMX; ++s) v[s] = lds[lslot<PAD>(i + s * Plan<N, RMX>::T, es)];
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

}  // namespace
}  // namespace ibdl
