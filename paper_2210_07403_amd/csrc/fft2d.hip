// FFT passes of two-dimensional grids (16 to 8192 points per axis), gfx950, wave64.
//
// The half spectra are kept transposed, [field][x mode][y] with the y lines contiguous and padded
// to nyp values (256 bytes beyond ny, so that consecutive x modes do not start on the same memory
// channel).  A block of the x passes takes R adjacent rows and writes, or reads, R adjacent y values
// per x mode (R * sizeof: 32 to 128 bytes), through the LDS that its transform uses anyway; the pass
// along y then reads and writes whole contiguous lines.  With the spectra row-major a y line of a
// 1024-point double-precision Stokes problem was a tile one line wide, 16 bytes of every 128-byte
// cache line of all rows, and lines over 1024 points needed two more passes over memory (a four-step
// transform); here one pass covers every length.
//
// Passes:  x axis  real <-> half spectrum, by an nx/2-point complex FFT of (x_2n + i x_2n+1) and the
//                  even/odd split.
//          lines   y axis: forward FFT of every input field, Fourier multiplier, inverse FFT of the
//                  output fields, in one kernel: the spectra never go back to memory in between.
//
// Measured against the row-major spectra (double precision, kernel medians): the 1024^2 Stokes pass along
// y 41 -> 17 us and its forward x pass 20.9 -> 12.0 us; the scalar pass 12.5 -> 8.6 us; on 4096^2 the
// three passes along y of one Stokes apply (five strided, the fused one, two strided) 968 -> 267 us,
// the forward x pass 295 -> 154 us over the active rows only.  What bounds them now: at 1024^2 and below
// the latency of the chain load, radix stages and their LDS exchanges, store, two lines to a CU; at 4096
// the same chain in a block that has its CU to itself (2.0 TB/s).
//
// Transforms whose lines are owned by at most one wave (T <= 64 threads) exchange through LDS
// without a workgroup barrier; longer ones alternate between two LDS buffers where they fit, one
// barrier per exchange.
#include "fft_core.h"
#include "kernels.h"

namespace ibdl {
namespace {

constexpr int kLds = 163840;      // LDS of a gfx950 workgroup
constexpr int kLdsHalf = 81920;   // two workgroups per CU

// ------------------------------------------------------------------ x axis
// Rows of M = nx / 2 complex values, T = M / RMX threads each, R rows per block.  LDS row stride: at
// least the padded exchange line and M + 1 modes, offset so that the R rows' accesses of one mode
// fall into different banks.
template <typename TR, int M> struct X2 {
  static constexpr int SZ = (int)sizeof(cplx<TR>);
  static constexpr int RMX = M < 8 ? M : (sizeof(TR) == 4 && M >= 2048 ? 16 : 8);
  static constexpr int T = M / RMX;
  static constexpr int BASE = (pad_len(M) + 1 + 31) / 32 * 32;
  static constexpr int BANKS = 256 / SZ;   // values per sweep of the 64 banks
  static constexpr int stride(int lr) { return BASE + (BANKS >> lr); }
  static constexpr int fits(int lr) { return (T << lr) <= 1024 && (stride(lr) << lr) * SZ <= kLds; }
  static constexpr int LMAX = fits(4) ? 4 : fits(3) ? 3 : fits(2) ? 2 : fits(1) ? 1 : 0;
  static constexpr int BLK = T << LMAX;
  // default rows per block: whole 128-byte lines of the spectra while two blocks of 512 threads share a
  // CU, else half lines (fewer where that leaves CUs without a block: rows_log2)
  static constexpr int want(int lr) {
    return lr > 0 && ((SZ << lr) > 128 || (T << lr) > 512 || (stride(lr) << lr) * SZ > kLdsHalf) ? want(lr - 1) : lr;
  }
  static constexpr int LDEF0 = want(LMAX);
  static constexpr int LDEF = (SZ << LDEF0) < 64 && (SZ << LMAX) >= 64 ? (LDEF0 + 1 < LMAX ? LDEF0 + 1 : LMAX) : LDEF0;
};

// forward: block (field f, rows y0 .. y0 + R - 1); TI: element type of the input rows (float rows
// widened on load for a double transform)
template <typename T, int M, typename TI>
__device__ __forceinline__ void r2c_block(const TI* __restrict__ in, cplx<T>* __restrict__ out, int ny, int nby, int lr,
                                          const cplx<T>* __restrict__ tw, const cplx<T>* __restrict__ st,
                                          const Rows2& rw, unsigned pitch, int64_t fs, int id) {
  using C = cplx<T>;
  using X = X2<T, M>;
  constexpr int RMX = X::RMX, TT = X::T;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  const int tid = threadIdx.x, R = 1 << lr, LS = X::stride(lr);
  const int f = id / nby, rb = id - f * nby;
  const int y0 = (rw.lo & ~(R - 1)) + (rb << lr);
  const int row = tid / TT, i = tid - row * TT, y = y0 + row;
  const bool live = y >= rw.lo && y <= rw.hi;
  const int64_t grow = (int64_t)f * ny + y;
  const cplx<TI>* src = reinterpret_cast<const cplx<TI>*>(in) + grow * M;
  C v[1][RMX];
  {
    bool on[RMX];
    if (rw.seg && live) {
      const unsigned long long* sg = rw.seg + (rw.seg_per_field ? grow : (int64_t)y) * rw.seg_words;
      if (rw.seg_words == 1) {
        const unsigned long long m = sg[0];
#pragma unroll
        for (int s = 0; s < RMX; ++s) on[s] = (m >> ((i + s * TT) >> rw.seg_log2)) & 1ull;
      } else {
        unsigned long long m[RMX];
#pragma unroll
        for (int s = 0; s < RMX; ++s) m[s] = sg[(i + s * TT) >> (rw.seg_log2 + 6)];
#pragma unroll
        for (int s = 0; s < RMX; ++s) on[s] = (m[s] >> (((i + s * TT) >> rw.seg_log2) & 63)) & 1ull;
      }
    } else {
#pragma unroll
      for (int s = 0; s < RMX; ++s) on[s] = live;
    }
#pragma unroll
    for (int s = 0; s < RMX; ++s) {
      v[0][s] = mk<C>(0, 0);
      if (on[s]) {
        const cplx<TI> x = src[i + s * TT];
        v[0][s] = mk<C>((T)x.x, (T)x.y);
      }
    }
    if (rw.sub && live && f >= rw.sub_f0 && f < rw.sub_f0 + rw.nsub) {   // minus a dense forcing
      const C* sub = static_cast<const C*>(rw.sub) + ((int64_t)(f - rw.sub_f0) * ny + y) * M;
#pragma unroll
      for (int s = 0; s < RMX; ++s) v[0][s] = csub(v[0][s], sub[i + s * TT]);
    }
  }
  C* line = lds + row * LS;
  C w0[RMX];
  int par = 0;
  fft_multi<M, false, 1, RMX, 1>(v, i, line, 0, par, st, w0);
  line_sync<TT>();
#pragma unroll
  for (int s = 0; s < RMX; ++s) line[i + s * TT] = v[0][s];
  // even/odd split, R adjacent threads taking the R rows of one mode
  const int r = tid & (R - 1), k0 = tid >> lr;
  C wk[RMX];
#pragma unroll
  for (int j = 0; j < RMX; ++j) wk[j] = tw[k0 + j * TT];
  __syncthreads();
  const C* z = lds + r * LS;
  const unsigned o0 = (unsigned)(y0 + r);
  out += f * fs;
#pragma unroll
  for (int j = 0; j < RMX; ++j) {
    const int k = k0 + j * TT;
    const C zk = z[k], zm = z[k == 0 ? 0 : M - k];
    const C E = mk<C>((zk.x + zm.x) * (T)0.5, (zk.y - zm.y) * (T)0.5);
    const C O = mk<C>((zk.y + zm.y) * (T)0.5, -(zk.x - zm.x) * (T)0.5);
    at(out, (o0 + (unsigned)k * pitch) * (unsigned)sizeof(C)) = cadd(E, cmul(wk[j], O));
    if (k == 0) at(out, (o0 + (unsigned)M * pitch) * (unsigned)sizeof(C)) = mk<C>(zk.x - zk.y, (T)0);
  }
}

template <typename T, int M, typename TI>
__global__ __launch_bounds__((X2<T, M>::BLK)) void k2_x_r2c(const TI* __restrict__ in, cplx<T>* __restrict__ out,
                                                            int ny, int nby, int lr, const cplx<T>* __restrict__ tw,
                                                            const cplx<T>* __restrict__ st,
                                                            Rows2 rw, unsigned pitch, int64_t fs) {
  // neighbouring row blocks on one XCD: they share the cache lines of the transposed spectra
  r2c_block<T, M, TI>(in, out, ny, nby, lr, tw, st, rw, pitch, fs, xcd_chunk((int)blockIdx.x, (int)gridDim.x));
}

// inverse: rows lo .. hi of the nfields output fields
template <typename T, int M>
__device__ __forceinline__ void c2r_block(const cplx<T>* __restrict__ in, T* __restrict__ out, int ny, int nby, int lr,
                                          const cplx<T>* __restrict__ tw, const cplx<T>* __restrict__ st,
                                          const Rows2& rw, unsigned pitch, int64_t fs, int id) {
  using C = cplx<T>;
  using X = X2<T, M>;
  constexpr int RMX = X::RMX, TT = X::T;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  const int tid = threadIdx.x, R = 1 << lr, LS = X::stride(lr);
  const int f = id / nby, rb = id - f * nby;
  const int y0 = (rw.lo & ~(R - 1)) + (rb << lr);
  {
    const int r = tid & (R - 1), k0 = tid >> lr;
    const unsigned o0 = (unsigned)(y0 + r);
    in += f * fs;
    C ld[RMX], last = mk<C>(0, 0);
#pragma unroll
    for (int j = 0; j < RMX; ++j) ld[j] = at(in, (o0 + (unsigned)(k0 + j * TT) * pitch) * (unsigned)sizeof(C));
    if (tid < R) last = at(in, (o0 + (unsigned)M * pitch) * (unsigned)sizeof(C));
    C* z = lds + r * LS;
#pragma unroll
    for (int j = 0; j < RMX; ++j) z[k0 + j * TT] = ld[j];
    if (tid < R) z[M] = last;
  }
  const int row = tid / TT, i = tid - row * TT, y = y0 + row;
  C wk[RMX];
#pragma unroll
  for (int s = 0; s < RMX; ++s) wk[s] = tw[i + s * TT];
  __syncthreads();
  // Z'_k = (X_k + conj X_{M-k}) + i conj(W^k) (X_k - conj X_{M-k})
  C* line = lds + row * LS;
  C v[1][RMX];
#pragma unroll
  for (int s = 0; s < RMX; ++s) {
    const int k = i + s * TT;
    const C a = line[k], b = line[M - k];
    v[0][s] = cadd(mk<C>(a.x + b.x, a.y - b.y), cmul(mk<C>(wk[s].y, wk[s].x), mk<C>(a.x - b.x, a.y + b.y)));
  }
  C w0[RMX];
  int par = 0;
  fft_multi<M, true, 1, RMX, 1>(v, i, line, 0, par, st, w0);
  if (y >= rw.lo && y <= rw.hi) {
    C* dst = reinterpret_cast<C*>(out) + ((int64_t)f * ny + y) * M;
#pragma unroll
    for (int s = 0; s < RMX; ++s) dst[i + s * TT] = v[0][s];
  }
}

template <typename T, int M>
__global__ __launch_bounds__((X2<T, M>::BLK)) void k2_x_c2r(const cplx<T>* __restrict__ in, T* __restrict__ out,
                                                            int ny, int nby, int lr, const cplx<T>* __restrict__ tw,
                                                            const cplx<T>* __restrict__ st,
                                                            Rows2 rw, unsigned pitch, int64_t fs) {
  c2r_block<T, M>(in, out, ny, nby, lr, tw, st, rw, pitch, fs, xcd_chunk((int)blockIdx.x, (int)gridDim.x));
}

// ------------------------------------------------------------------ y axis
// What a pass along y does between the forward transforms of its NI input fields and the inverse
// transforms of its NO output fields:
//   L_SCALAR  u^ = a (sum_f c_f F^_f) / (c2 sigma - c0), c_f = i k~_d (FK_DX, FK_DY) or 1 (FK_MASS);
//             0 where the denominator vanishes (mean-zero inverse)
//   L_STOKES  with ell = -sigma, lam = c2 ell + c0, P^ = I - k~ k~^T / ell (1/ell, 1/lam read as 0
//             where they vanish), s = (A11 + A22)/2, v_i = sum_j i k~_j A_ij:
//             u^ = a [ i k~ s^/ell + (1/lam) P^ (G^ + mu v^) ]
//   L_PRESS   p^ = a [ -i k~_j G^_j + mu k~_i k~_j A^_ij + (c2 sigma - c0) s^ ] / ell
//   L_GRAD    one input F: i k~_x g F^, i k~_y g F^ and g F^, g = a / (c2 sigma - c0)
//   L_ADJ     the transpose of L_STOKES: two components in, the duals of A11, A12, A22 (G1, G2) out
// Stokes inputs are (A11, A12, A22), then or only (G1, G2).
//   L_FWD, L_INV  the transforms of one field alone
enum LineKind { L_SCALAR, L_STOKES, L_PRESS, L_GRAD, L_ADJ, L_FWD, L_INV };

template <typename T> struct Mode {   // symbols of one (x, y) mode
  T kx, ky, sig;
};
// whether a pass needs k~ along y (a single scalar input is an FK_MASS field)
constexpr bool line_needs_k(int kind, int ni) { return !(kind == L_SCALAR && ni == 1); }
template <typename T> __device__ __forceinline__ T inv0(T v) { return v == (T)0 ? (T)0 : recip(v); }
template <typename C> __device__ __forceinline__ C mul_i(C a) { return mk<C>(-a.y, a.x); }

// all outputs of one mode from all inputs
template <int KIND, int NI, int NO, typename T, typename C = cplx<T>>
__device__ __forceinline__ void mode_mult(const MultDesc& md, const Mode<T>& m, const C (&x)[NI], C (&y)[NO]) {
  const T a = (T)(md.alpha * md.sc), c2 = (T)md.c2, c0 = (T)md.c0, mu = (T)md.mu;
  if constexpr (KIND == L_SCALAR || KIND == L_GRAD) {
    const T den = c2 * m.sig - c0;
    const T g = den == (T)0 ? (T)0 : a * recip(den);
    if constexpr (KIND == L_GRAD) {
      y[0] = mul_ir(x[0], g * m.kx);
      if constexpr (NO > 1) y[1] = mul_ir(x[0], g * m.ky);
      if constexpr (NO > 2) y[2] = cscale(x[0], g);
    } else {
      if constexpr (NI == 1) {
        y[0] = cscale(x[0], g);
        return;
      }
      y[0] = mk<C>(0, 0);
#pragma unroll
      for (int f = 0; f < NI; ++f) {
        const int fk = md.fk[f];
        y[0] = cadd(y[0], fk == FK_MASS ? cscale(x[f], g) : mul_ir(x[f], g * (fk == FK_DX ? m.kx : m.ky)));
      }
    }
  } else {
    const T ell = -m.sig, il = inv0(ell), lam = c2 * ell + c0, is = inv0(lam);
    if constexpr (KIND == L_ADJ) {
      const C kF = cadd(cscale(x[0], m.kx), cscale(x[1], m.ky));
      const C p0 = csub(x[0], cscale(kF, m.kx * il)), p1 = csub(x[1], cscale(kF, m.ky * il));
      const T h = (T)-0.5 * a * il, s = -a * mu * is;
      y[0] = mul_i(cadd(cscale(kF, h), cscale(p0, s * m.kx)));
      if constexpr (NO > 1) y[1] = mul_i(cadd(cscale(p0, s * m.ky), cscale(p1, s * m.kx)));
      if constexpr (NO > 2) y[2] = mul_i(cadd(cscale(kF, h), cscale(p1, s * m.ky)));
      if constexpr (NO > 3) y[3] = cscale(p0, a * is);
      if constexpr (NO > 4) y[4] = cscale(p1, a * is);
    } else {
      constexpr bool A = NI != 2;            // dipole fields present
      constexpr int G = NI == 2 ? 0 : 3;     // first single-layer field
      constexpr bool HG = NI == 2 || NI == 5;
      if constexpr (KIND == L_PRESS) {
        const T lh = (T)0.5 * (c2 * m.sig - c0), t = a * il;
        C p = mk<C>(0, 0);
        if constexpr (A) {
          p = cadd(cscale(x[0], t * (mu * m.kx * m.kx + lh)), cscale(x[1], t * ((T)2 * mu * m.kx * m.ky)));
          p = cadd(p, cscale(x[2], t * (mu * m.ky * m.ky + lh)));
        }
        if constexpr (HG) p = csub(p, mul_i(cadd(cscale(x[G], t * m.kx), cscale(x[G + 1], t * m.ky))));
        y[0] = p;
      } else {
        C F0 = mk<C>(0, 0), F1 = mk<C>(0, 0);
        if constexpr (A) {
          F0 = mul_ir(cadd(cscale(x[0], m.kx), cscale(x[1], m.ky)), mu);
          F1 = mul_ir(cadd(cscale(x[1], m.kx), cscale(x[2], m.ky)), mu);
        }
        if constexpr (HG) {
          F0 = cadd(F0, x[G]);
          F1 = cadd(F1, x[G + 1]);
        }
        const C kF = cadd(cscale(F0, m.kx), cscale(F1, m.ky));
        y[0] = cscale(csub(F0, cscale(kF, m.kx * il)), a * is);
        y[1] = cscale(csub(F1, cscale(kF, m.ky * il)), a * is);
        if constexpr (A) {
          const C s = mul_ir(cadd(x[0], x[2]), (T)0.5 * a * il);
          y[0] = cadd(y[0], cscale(s, m.kx));
          y[1] = cadd(y[1], cscale(s, m.ky));
        }
      }
    }
  }
}

// Elements per thread of a y line: 8 for one field.  Passes that hold several fields at once take 4 in
// double (five fields at 4 take 80 registers), in float from 2048 points on, where a block of 512 or
// 1024 threads leaves 128 registers.  Double lines of 2048 and 4096 points take 8: 2048 lines of 2048
// points, five fields and two: 82 us with 4 on 512 threads, 62 with 8 on 256 threads and twiddles read as
// they are used; lines of 1024 with 8: 24 us, with 4: 17.  Registers spill all the same, mostly in the packed
// block (line_packs): with five fields 205 of them at 2048 points (6 without it) and 208 at 4096 (none).
// Lines of 8192 points need 8 to fit 1024 threads.
template <typename T> constexpr int line_rmx(int N, int nmax) {
  if (N <= 8) return N;
  if (nmax == 1 || N < 64) return 8;
  if (N == 8192) return 8;
  if (sizeof(T) == 8 && N >= 2048) return 8;
  return sizeof(T) == 8 || N >= 2048 ? 4 : 8;
}
template <typename T, int N, int NI, int NO> struct LineShape {
  static constexpr int NM = NI > NO ? NI : NO;
  static constexpr int RMX = line_rmx<T>(N, NM);
  static constexpr int T_ = N / RMX;
  static constexpr int SZ = (int)sizeof(cplx<T>);
  static constexpr int LP = pad_len(N);
  // waves per SIMD that the register bound aims at: the five-field 4096-point double pass keeps its 160
  // registers of data and one block per CU (measured 275 us a launch on 4096^2 with two exchange
  // buffers, 312 with one; 4 elements per thread on 1024 threads of 128 registers: 355; 16 on 256: 472)
  static constexpr bool ALONE = sizeof(T) == 8 && N == 4096 && NM > 3;
  // Blocks of 512 threads or more: registers are what bounds the waves per SIMD, so the second
  // transform reads its twiddles again (from cache) instead of keeping the first one's, and the
  // symbols are read as they are used.
  static constexpr bool D2048 = sizeof(T) == 8 && N == 2048 && NM > 1;   // 8 elements on 256 threads
  static constexpr bool LEAN = T_ >= 512 || D2048;
  // Double passes of 4096 points with two or three fields get 128 registers for 64 or 96 of data and spill in
  // every block (one field in, three out 318 of them, three in and two out 521, three in and one out 574):
  // applies on 4096^2 with them take 451, 501 and 637 us, with one field in and out 153.
  static constexpr int MINW = D2048 ? 2 : !LEAN ? 1 : ALONE ? 2 : 4;
  // two exchange buffers per line where two blocks then still share a CU, or where the block has
  // the CU to itself anyway
  static constexpr int NBUF =
      T_ <= 64 ? 1 : (2 * LP * SZ <= kLdsHalf || ((ALONE || (T_ == 1024 && NM > 1)) && 2 * LP * SZ <= kLds) ? 2 : 1);
  static constexpr int W = T_ >= 256 ? 1 : 256 / T_;   // most lines per block
  static constexpr int BLK = T_ >= 256 ? T_ : 256;
  // Lines of 8192 points with several fields (more than three in float): the fields' registers would
  // spill, so the transforms and the multiplier run as separate passes (7 -> 21 field passes over
  // memory for a Stokes apply)
  static constexpr bool SPLIT = N == 8192 && NM > (sizeof(T) == 8 ? 1 : 3);
  static_assert(LP * NBUF * SZ <= kLds, "y line: LDS over budget");
};

// The lines kx = 0 and kx = nx / 2 are spectra of real data: real along y, like every product with the
// symbols (k~ vanishes at 0 and at the half), so one complex line a + i b carries both, and nx / 2 lines
// are left of nx / 2 + 1.  That line more was a block more than the CUs hold at once, a whole round for
// itself: five fields and two, FP64, 513 lines of 1024 points 22.4 us, 2049 of 4096 275 us, with the two
// packed 17.2 and 267; one field, 2049 of 4096, 67 and 63.  Where a line has 256 threads or more; with
// fewer a CU holds enough blocks.
//
// half_swap: the transform Z of a + i b, in place, to a^ in slots 0 < k < N/2 and b^ in the slots N - k
// (a^ + i b^ of the real modes stays in slots 0 and N/2); with JOIN back.
template <int N, int RMX, bool JOIN, typename C>
__device__ __forceinline__ void half_swap(C (&v)[RMX], int i, C* lds) {
  constexpr int TT = N / RMX;
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
#pragma unroll
  for (int s = 0; s < RMX; ++s) lds[pad_at(i) + pad_len(s * TT)] = v[s];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < RMX; ++s) {
    if ((s == 0 || s == RMX / 2) && i == 0) continue;
    const C a = v[s], m = lds[pad_at(N - (i + s * TT))];
    if constexpr (JOIN) v[s] = s < RMX / 2 ? mk<C>(a.x - m.y, a.y + m.x) : mk<C>(m.x + a.y, a.x - m.y);
    else v[s] = cscale(s < RMX / 2 ? mk<C>(a.x + m.x, a.y - m.y) : mk<C>(m.y + a.y, a.x - m.x), decltype(a.x)(0.5));
  }
}
template <int N, int KIND, int T_> constexpr bool line_packs() {
  return T_ >= 256 && KIND != L_FWD && KIND != L_INV;
}

// PACK: the block of lines 0 and jh
template <typename T, int N, int NI, int NO, int KIND, bool PACK>
__device__ __forceinline__ void lines_block(cplx<T>* __restrict__ data, const MultDesc& md,
                                            const cplx<T>* __restrict__ tw, int W, const RowMask& rm, int bx) {
  using C = cplx<T>;
  using L = LineShape<T, N, NI, NO>;
  constexpr int RMX = L::RMX, TT = L::T_, NBUF = L::NBUF;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, c = tid / TT, i = tid - c * TT;
  C* lds = reinterpret_cast<C*>(smem) + c * (NBUF * L::LP);
  const int kx = bx * W + c;
  const bool valid = kx < md.nxh;
  const int jx = valid ? kx : 0, jh = md.nxh - 1;
  const unsigned fs = (unsigned)md.nxh * (unsigned)md.nyp;
  const unsigned b0 = ((unsigned)jx * (unsigned)md.nyp + (unsigned)i) * (unsigned)sizeof(C);
  constexpr unsigned step = TT * (unsigned)sizeof(C);
  const unsigned fsb = fs * (unsigned)sizeof(C);
  const T* sgl = static_cast<const T*>(md.sig[1]);
  const T* ktl = static_cast<const T*>(md.kt[1]);
  const T sigx = static_cast<const T*>(md.sig[0])[jx], kxs = static_cast<const T*>(md.kt[0])[jx];
  const unsigned bh = ((unsigned)jh * (unsigned)md.nyp + (unsigned)i) * (unsigned)sizeof(C);
  // a slot of the packed line that holds a mode of line jh (half_swap), and its y mode
  auto half = [&](int s) { return PACK && s >= RMX / 2 && i + s * TT != N / 2; };
  auto ymode = [&](int s) { return half(s) ? N - (i + s * TT) : i + s * TT; };
  auto load = [&](C (&v)[RMX], int f) {
#pragma unroll
    for (int s = 0; s < RMX; ++s) {
      const int y = i + s * TT;
      const bool on = valid && (!rm.load || (y >= rm.lo && y <= rm.hi));
      v[s] = on ? at(data, (unsigned)f * fsb + b0 + s * step) : mk<C>(0, 0);
      if constexpr (PACK) v[s].y = on ? at(data, (unsigned)f * fsb + bh + s * step).x : (T)0;
    }
  };
  auto store = [&](const C (&v)[RMX], int f) {
#pragma unroll
    for (int s = 0; s < RMX; ++s) {
      const int y = i + s * TT;
      if (valid && (!rm.store || (y >= rm.lo && y <= rm.hi))) {
        C a = v[s];
        if constexpr (PACK) {
          at(data, (unsigned)f * fsb + bh + s * step) = mk<C>(a.y, (T)0);
          a.y = (T)0;
        }
        at(data, (unsigned)f * fsb + b0 + s * step) = a;
      }
    }
  };
  C w0[RMX];
  int par = 0;
  const C* tw2 = tw;   // the inverse transforms' table: with LEAN a copy the compiler cannot identify with tw
  if constexpr (L::LEAN) asm volatile("" : "+s"(tw2));
  C v[NI][RMX];
#pragma unroll
  for (int f = 0; f < NI; ++f) load(v[f], f);
  if constexpr (KIND == L_FWD || KIND == L_INV) {   // one transform, nothing else
    fft_multi<N, KIND == L_INV, 1, RMX, NBUF, L::LEAN>(v, i, lds, L::LP, par, tw, w0);
    store(v[0], 0);
  } else {
    T sg[RMX], ks[RMX];
    if constexpr (!L::LEAN) {
#pragma unroll
      for (int s = 0; s < RMX; ++s) {
        sg[s] = sgl[ymode(s)];
        ks[s] = line_needs_k(KIND, NI) ? ktl[ymode(s)] : (T)0;
      }
    }
    fft_multi<N, false, NI, RMX, NBUF, L::LEAN>(v, i, lds, L::LP, par, tw, w0);
    if constexpr (PACK) {
#pragma unroll
      for (int f = 0; f < NI; ++f) half_swap<N, RMX, false>(v[f], i, lds);
      __syncthreads();
    }
    __builtin_amdgcn_sched_barrier(0);
    C u[NO][RMX];
#pragma unroll
    for (int s = 0; s < RMX; ++s) {
      if constexpr (L::LEAN) {
        __builtin_amdgcn_sched_barrier(0);
        sg[s] = sgl[ymode(s)];
        ks[s] = line_needs_k(KIND, NI) ? ktl[ymode(s)] : (T)0;
      }
      Mode<T> m{kxs, ks[s], sigx + sg[s]};
      if constexpr (PACK) {
        if (half(s)) {
          m.kx = static_cast<const T*>(md.kt[0])[jh];
          m.sig = static_cast<const T*>(md.sig[0])[jh] + sg[s];
        }
      }
      C x[NI], y[NO];
#pragma unroll
      for (int f = 0; f < NI; ++f) x[f] = v[f][s];
      mode_mult<KIND, NI, NO, T>(md, m, x, y);
#pragma unroll
      for (int o = 0; o < NO; ++o) u[o][s] = y[o];
      if (PACK && (s == 0 || s == RMX / 2)) {
        if (i == 0) {   // the packed real modes: real part from line 0's symbols, imaginary part from line jh's
          m.kx = static_cast<const T*>(md.kt[0])[jh];
          m.sig = static_cast<const T*>(md.sig[0])[jh] + sg[s];
          mode_mult<KIND, NI, NO, T>(md, m, x, y);
#pragma unroll
          for (int o = 0; o < NO; ++o) u[o][s].y = y[o].y;
        }
      }
    }
    if constexpr (PACK) {
#pragma unroll
      for (int o = 0; o < NO; ++o) half_swap<N, RMX, true>(u[o], i, lds);
      __syncthreads();
    }
    fft_multi<N, true, NO, RMX, NBUF, L::LEAN>(u, i, lds, L::LP, par, tw2, w0);
#pragma unroll
    for (int o = 0; o < NO; ++o) store(u[o], o);
  }
}

template <typename T, int N, int NI, int NO, int KIND>
__global__ __launch_bounds__((LineShape<T, N, NI, NO>::BLK), (LineShape<T, N, NI, NO>::MINW)) void k2_lines(cplx<T>* __restrict__ data, MultDesc md,
                                                                         const cplx<T>* __restrict__ tw, int W,
                                                                         int64_t bstride, RowMask rm) {
  data += (int64_t)blockIdx.y * bstride;   // problem of a batch
  if constexpr (line_packs<N, KIND, LineShape<T, N, NI, NO>::T_>()) {
    if (blockIdx.x == 0) {
      // (own copies of the pointers: the compiler would otherwise hold what both paths load for both)
      cplx<T>* d = data;
      const cplx<T>* t = tw;
      asm volatile("" : "+s"(d), "+s"(t));
      lines_block<T, N, NI, NO, KIND, true>(d, md, t, W, rm, 0);
      return;
    }
  }
  lines_block<T, N, NI, NO, KIND, false>(data, md, tw, W, rm, (int)blockIdx.x);
}

// the multiplier by itself, on transformed fields (LineShape::SPLIT)
template <typename T, int NI, int NO, int KIND>
__global__ __launch_bounds__(256) void k2_mult(cplx<T>* __restrict__ data, MultDesc md, int n) {
  using C = cplx<T>;
  const int e = (int)blockIdx.x * 256 + (int)threadIdx.x, jx = (int)blockIdx.y;
  if (e >= n) return;
  const int64_t fs = (int64_t)md.nxh * md.nyp, o0 = (int64_t)jx * md.nyp + e;
  const Mode<T> m{static_cast<const T*>(md.kt[0])[jx], static_cast<const T*>(md.kt[1])[e],
                  static_cast<const T*>(md.sig[0])[jx] + static_cast<const T*>(md.sig[1])[e]};
  C x[NI], y[NO];
#pragma unroll
  for (int f = 0; f < NI; ++f) x[f] = data[f * fs + o0];
  mode_mult<KIND, NI, NO, T>(md, m, x, y);
#pragma unroll
  for (int o = 0; o < NO; ++o) data[o * fs + o0] = y[o];
}

// ------------------------------------------------------------------ several grids in one launch
// The three passes of a batch's grid groups (one field, scalar multiplier), one launch per pass for all
// groups instead of one per group and pass: workgroup b takes block items[b].y of group items[b].x.
// A block holds 2,048 values whatever its line length, so the blocks are alike.  Launches of a few
// dozen blocks each, one behind the other, were what a batch of small grids spent its time on: 30
// problems on 128^2, 256^2 and 512^2 grids, FP64, nine launches 63 us, three launches 45.
constexpr int kGroupM0 = 32, kGroupM1 = 512, kGroupN1 = 1024;   // row lengths (complex), longest y line
template <int M, typename F> __device__ __forceinline__ void group_row(int m, F&& f) {
  if constexpr (M <= kGroupM1) {
    if (m == M) f(std::integral_constant<int, M>{});
    else group_row<2 * M>(m, f);
  }
}
template <typename T> constexpr int group_rows_log2(int m) { return m == 32 ? 6 : m == 64 ? 5 : m == 128 ? 4 : m == 256 ? 3 : 2; }

template <typename T, bool INV>
__global__ __launch_bounds__(256) void k2_x_groups(const Fft2Group* __restrict__ gd, const int2* __restrict__ items) {
  using C = cplx<T>;
  const int2 it = items[xcd_chunk((int)blockIdx.x, (int)gridDim.x)];
  const Fft2Group& g = gd[__builtin_amdgcn_readfirstlane(it.x)];
  const int id = __builtin_amdgcn_readfirstlane(it.y);
  const unsigned pitch = (unsigned)spec2_pitch<T>(g.ny);
  const int64_t fs = (int64_t)(g.m + 1) * pitch;
  group_row<kGroupM0>(g.m, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value, LR = group_rows_log2<T>(M);
    static_assert(M / 8 << LR == 256, "a block holds 2,048 values");
    const C* base = static_cast<const C*>(g.base);
    const C* st = static_cast<const C*>(g.twx);
    if constexpr (INV)
      c2r_block<T, M>(static_cast<const C*>(g.spec), static_cast<T*>(g.real), g.ny, g.nbx, LR, base, st, g.out, pitch, fs, id);
    else
      r2c_block<T, M, T>(static_cast<const T*>(g.real), static_cast<C*>(g.spec), g.ny, g.nbx, LR, base, st, g.in, pitch, fs, id);
  });
}

template <int N, typename F> __device__ __forceinline__ void group_line(int n, F&& f) {
  if constexpr (N <= kGroupN1) {
    if (n == N) f(std::integral_constant<int, N>{});
    else group_line<2 * N>(n, f);
  }
}
template <typename T>
__global__ __launch_bounds__(256) void k2_lines_groups(const Fft2Group* __restrict__ gd, const int2* __restrict__ items) {
  using C = cplx<T>;
  const int2 it = items[blockIdx.x];
  const Fft2Group& g = gd[__builtin_amdgcn_readfirstlane(it.x)];
  const int id = __builtin_amdgcn_readfirstlane(it.y), p = id / g.nbl;
  const int64_t fs = (int64_t)(g.m + 1) * spec2_pitch<T>(g.ny);
  group_line<16>(g.ny, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    using L = LineShape<T, N, 1, 1>;
    static_assert(L::W * L::T_ == 256 && !line_packs<N, L_SCALAR, L::T_>(), "a block of 256 threads");
    lines_block<T, N, 1, 1, L_SCALAR, false>(static_cast<C*>(g.spec) + p * fs, g.md, static_cast<const C*>(g.twy), L::W,
                                             RowMask(), id - p * g.nbl);
  });
}

template <typename F> void dispatch2(int n, F&& f) {
  switch (n) {
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    case 256: f(std::integral_constant<int, 256>{}); break;
    case 512: f(std::integral_constant<int, 512>{}); break;
    case 1024: f(std::integral_constant<int, 1024>{}); break;
    case 2048: f(std::integral_constant<int, 2048>{}); break;
    case 4096: f(std::integral_constant<int, 4096>{}); break;
    default: throw Error(-2, "unsupported FFT length " + std::to_string(n));
  }
}
template <typename F> void dispatch2_line(int n, F&& f) {
  if (n == 8192) f(std::integral_constant<int, 8192>{});
  else if (n < 16) throw Error(-2, "unsupported FFT length " + std::to_string(n));
  else dispatch2(n, f);
}

int log2_rows(int want, int ldef, int lmax) {
  if (want <= 0) return ldef;
  int l = 0;
  while (l < lmax && (2 << l) <= want) ++l;
  return l;
}

// Rows per block of an x pass (log2), T threads each: what the caller asks for, or the default, halved while
// that leaves CUs without a block and a block has more than a wave.  Single precision, one field, three passes: 4096 x 512 points 42 us with the default's 64
// blocks, 32 with 128, 29 with 256, 33 with 512; 2048 x 512 25.5, 20.5, 18.5, 20.4; 1024^2 18.4, 18.3, 17.2, 18.1.
int rows_log2(int rpb, int ldef, int lmax, int T, const Rows2& rw, int nf) {
  constexpr int64_t kCus = 256;
  int lr = log2_rows(rpb, ldef, lmax);
  if (rpb <= 0)
    while (lr > 0 && (T << lr) > 64 &&
           (int64_t)nf * (((rw.hi | ((1 << lr) - 1)) - (rw.lo & ~((1 << lr) - 1)) + 1) >> lr) < kCus) --lr;
  return lr;
}

void check_span(int64_t fs, int nf, size_t size) {
  if (fs * nf * (int64_t)size > (int64_t)UINT32_MAX)
    throw Error(-2, "2-D FFT pass: one problem's fields may not span 4 GiB");
}

template <typename T, typename TI>
void r2c_launch(const TI* in, cplx<T>* out, int nx, int ny, int nf, const Tw2<T>& tw, hipStream_t s, int rpb,
                const Rows2& rw) {
  if (nf < 1 || rw.hi < rw.lo) return;
  const int64_t fs = spec2_size<T>(nx, ny);
  check_span(fs, 1, sizeof(cplx<T>));
  dispatch2(nx / 2, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value;
    using X = X2<T, M>;
    const int lr = rows_log2(rpb, X::LDEF, X::LMAX, X::T, rw, nf), R = 1 << lr;
    const int nby = ((rw.hi | (R - 1)) - (rw.lo & ~(R - 1)) + 1) / R;
    hipLaunchKernelGGL((k2_x_r2c<T, M, TI>), dim3((unsigned)(nby * nf)), dim3(X::T << lr),
                       (size_t)(X::stride(lr) << lr) * sizeof(cplx<T>), s, in, out, ny, nby, lr, tw.base, tw.x, rw,
                       (unsigned)spec2_pitch<T>(ny), fs);
  });
  IBDL_LAUNCH_CHECK();
}

}  // namespace

template <typename T>
void fft2_x_r2c(const T* in, cplx<T>* out, int nx, int ny, int nf, const Tw2<T>& tw, hipStream_t s, int rpb,
                const Rows2& rw) {
  r2c_launch<T, T>(in, out, nx, ny, nf, tw, s, rpb, rw);
}

void fft2_x_r2c_widen(const float* in, cplx<double>* out, int nx, int ny, int nf, const Tw2<double>& tw, hipStream_t s,
                      int rpb, const Rows2& rw) {
  r2c_launch<double, float>(in, out, nx, ny, nf, tw, s, rpb, rw);
}

template <typename T>
void fft2_x_c2r(const cplx<T>* in, T* out, int nx, int ny, int nf, const Tw2<T>& tw, hipStream_t s, int rpb,
                const Rows2& rw) {
  if (nf < 1 || rw.hi < rw.lo) return;
  const int64_t fs = spec2_size<T>(nx, ny);
  check_span(fs, 1, sizeof(cplx<T>));
  dispatch2(nx / 2, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value;
    using X = X2<T, M>;
    const int lr = rows_log2(rpb, X::LDEF, X::LMAX, X::T, rw, nf), R = 1 << lr;
    const int nby = ((rw.hi | (R - 1)) - (rw.lo & ~(R - 1)) + 1) / R;
    hipLaunchKernelGGL((k2_x_c2r<T, M>), dim3((unsigned)(nby * nf)), dim3(X::T << lr),
                       (size_t)(X::stride(lr) << lr) * sizeof(cplx<T>), s, in, out, ny, nby, lr, tw.base, tw.x, rw,
                       (unsigned)spec2_pitch<T>(ny), fs);
  });
  IBDL_LAUNCH_CHECK();
}

template <typename T>
void fft2_lines(cplx<T>* data, int n, int no, const MultDesc& md, const Tw2<T>& tw, hipStream_t s, int batch,
                int64_t bstride, int w, const RowMask& rm) {
  if (batch < 1) return;
  check_span((int64_t)md.nxh * md.nyp, std::max(std::max(md.nc, no), 1), sizeof(cplx<T>));
  dispatch2_line(n, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    auto go = [&](auto nic, auto noc, auto kc) {
      constexpr int NI = decltype(nic)::value, NO = decltype(noc)::value, KIND = decltype(kc)::value;
      auto line = [&](auto nic1, auto noc1, auto kc1, int count, int64_t stride, const RowMask& mask) {
        constexpr int I = decltype(nic1)::value, O = decltype(noc1)::value;
        using L = LineShape<T, N, I, O>;
        int W = 1;
        while (2 * W <= (w <= 0 || w > L::W ? L::W : w)) W *= 2;
        const int nl = md.nxh - (line_packs<N, decltype(kc1)::value, L::T_>() ? 1 : 0);
        const dim3 grid((unsigned)((nl + W - 1) / W), (unsigned)count);
        hipLaunchKernelGGL((k2_lines<T, N, I, O, decltype(kc1)::value>), grid, dim3(W * L::T_),
                           (size_t)W * L::NBUF * L::LP * sizeof(cplx<T>), s, data, md,
                           tw.y[L::NM > 1 ? 1 : 0], W, stride, mask);
      };
      if constexpr (LineShape<T, N, NI, NO>::SPLIT) {
        if (batch != 1) throw Error(-2, "2-D line pass: batches hold lines of up to 1024 points");
        using one = std::integral_constant<int, 1>;
        const int64_t fs = (int64_t)md.nxh * md.nyp;
        RowMask in = rm, out = rm;
        in.store = 0;
        out.load = 0;
        line(one{}, one{}, std::integral_constant<int, L_FWD>{}, NI, fs, in);
        hipLaunchKernelGGL((k2_mult<T, NI, NO, KIND>), dim3((unsigned)((n + 255) / 256), (unsigned)md.nxh), dim3(256), 0, s,
                           data, md, n);
        line(one{}, one{}, std::integral_constant<int, L_INV>{}, NO, fs, out);
      } else {
        line(nic, noc, kc, batch, bstride, rm);
      }
    };
    using std::integral_constant;
#define IBDL_LINE(ni, no_, kind) go(integral_constant<int, ni>{}, integral_constant<int, no_>{}, integral_constant<int, kind>{})
    if (md.mode == 1 && md.nc == 1 && no == 2) IBDL_LINE(1, 2, L_GRAD);
    else if (md.mode == 1 && md.nc == 1 && no == 3) IBDL_LINE(1, 3, L_GRAD);
    else if (md.mode == 2 && md.stokes && md.nc == 2 && no == 3) IBDL_LINE(2, 3, L_ADJ);
    else if (md.mode == 2 && md.stokes && md.nc == 2 && no == 5) IBDL_LINE(2, 5, L_ADJ);
    else if (md.mode == 3 && md.stokes && md.nc == 3 && no == 1) IBDL_LINE(3, 1, L_PRESS);
    else if (md.mode == 3 && md.stokes && md.nc == 5 && no == 1) IBDL_LINE(5, 1, L_PRESS);
    else if (md.mode != 0) throw Error(-2, "2-D line pass: unsupported transposed multiplier");
    else if (!md.stokes && no == 1 && md.nc == 1 && md.fk[0] == FK_MASS) IBDL_LINE(1, 1, L_SCALAR);
    else if (!md.stokes && no == 1 && md.nc == 2) IBDL_LINE(2, 1, L_SCALAR);
    else if (!md.stokes && no == 1 && md.nc == 3) IBDL_LINE(3, 1, L_SCALAR);
    else if (md.stokes && no == 2 && md.nc == 2) IBDL_LINE(2, 2, L_STOKES);
    else if (md.stokes && no == 2 && md.nc == 3) IBDL_LINE(3, 2, L_STOKES);
    else if (md.stokes && no == 2 && md.nc == 5) IBDL_LINE(5, 2, L_STOKES);
    else throw Error(-2, "2-D line pass: unsupported multiplier / field count");
#undef IBDL_LINE
  });
  IBDL_LAUNCH_CHECK();
}

// A grid can take part in the merged passes when its rows and lines have merged forms and a block's
// rows, 4096 / nx of them, do not reach past the grid.
bool fft2_groups_fit(int nx, int ny) {
  return nx >= 2 * kGroupM0 && nx <= 2 * kGroupM1 && ny >= 16 && ny <= kGroupN1 && 4096 / nx <= ny;
}

template <typename T>
void fft2_group_set(Fft2Group& g, T* real, cplx<T>* spec, int nx, int ny, int np, const Tw2<T>& tw) {
  if (!fft2_groups_fit(nx, ny)) throw Error(-2, "merged 2-D passes: unsupported grid");
  check_span(spec2_size<T>(nx, ny), 1, sizeof(cplx<T>));
  g.real = real;
  g.spec = spec;
  g.ny = ny;
  g.m = nx / 2;
  g.np = np;
  g.nbx = ny / (4096 / nx);
  const int W = 256 / (ny / 8);
  g.nbl = (g.m + 1 + W - 1) / W;
  g.base = tw.base;
  g.twx = tw.x;
  g.twy = tw.y[0];
}

template <typename T>
void fft2_groups(const Fft2Group* host, const Fft2Group* dev, int ng, const int2* items, int nx_items, int ny_items,
                 hipStream_t s) {
  if (nx_items <= 0 || ny_items <= 0) return;
  size_t ldx = 0, ldy = 0;
  for (int k = 0; k < ng; ++k) {
    dispatch2(host[k].m, [&](auto Mc) {
      constexpr int M = decltype(Mc)::value;
      if constexpr (M >= kGroupM0 && M <= kGroupM1) {
        constexpr int LR = group_rows_log2<T>(M);
        ldx = std::max(ldx, (size_t)(X2<T, M>::stride(LR) << LR) * sizeof(cplx<T>));
      }
    });
    dispatch2_line(host[k].ny, [&](auto Nc) {
      using L = LineShape<T, decltype(Nc)::value, 1, 1>;
      ldy = std::max(ldy, (size_t)L::W * L::NBUF * L::LP * sizeof(cplx<T>));
    });
  }
  hipLaunchKernelGGL((k2_x_groups<T, false>), dim3((unsigned)nx_items), dim3(256), ldx, s, dev, items);
  hipLaunchKernelGGL((k2_lines_groups<T>), dim3((unsigned)ny_items), dim3(256), ldy, s, dev, items + nx_items);
  hipLaunchKernelGGL((k2_x_groups<T, true>), dim3((unsigned)nx_items), dim3(256), ldx, s, dev, items);
  IBDL_LAUNCH_CHECK();
}

namespace {
template <typename T> struct TableLens { int x, y0, y1; };
template <typename T> TableLens<T> table_lens(int nx, int ny) {
  TableLens<T> l{};
  dispatch2(nx / 2, [&](auto Mc) { l.x = stage_len<decltype(Mc)::value, X2<T, decltype(Mc)::value>::RMX>(); });
  dispatch2_line(ny, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    l.y0 = stage_len<N, line_rmx<T>(N, 1)>();
    l.y1 = stage_len<N, line_rmx<T>(N, 2)>();
  });
  return l;
}
}  // namespace

template <typename T> size_t fft2_table_len(int nx, int ny) {
  const TableLens<T> l = table_lens<T>(nx, ny);
  return (size_t)l.x + l.y0 + l.y1 + 1;
}

template <typename T>
Tw2<T> fft2_tables(int nx, int ny, const cplx<T>* twx, const cplx<T>* twy, cplx<T>* dst, hipStream_t s) {
  using C = cplx<T>;
  const TableLens<T> l = table_lens<T>(nx, ny);
  C* x = dst;
  C* y[2] = {dst + l.x, dst + l.x + l.y0};
  auto blocks = [](int n) { return dim3((unsigned)((n + 255) / 256)); };
  dispatch2(nx / 2, [&](auto Mc) {
    constexpr int M = decltype(Mc)::value;
    if (l.x > 0) hipLaunchKernelGGL((k_stages<M, X2<T, M>::RMX, C>), blocks(l.x), dim3(256), 0, s, x, twx, 2);
  });
  dispatch2_line(ny, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    if (l.y0 > 0) hipLaunchKernelGGL((k_stages<N, line_rmx<T>(N, 1), C>), blocks(l.y0), dim3(256), 0, s, y[0], twy, 1);
    if (l.y1 > 0) hipLaunchKernelGGL((k_stages<N, line_rmx<T>(N, 2), C>), blocks(l.y1), dim3(256), 0, s, y[1], twy, 1);
  });
  IBDL_LAUNCH_CHECK();
  Tw2<T> t;
  t.base = twx;
  t.x = x;
  t.y[0] = y[0];
  t.y[1] = y[1];
  return t;
}

template <typename T> int fft2_rows_max(int nx) {
  int r = 1;
  dispatch2(nx / 2, [&](auto Mc) { r = 1 << X2<T, decltype(Mc)::value>::LMAX; });
  return r;
}

template <typename T> int fft2_lines_max(int n, int nmax) {
  int r = 1;
  dispatch2_line(n, [&](auto Nc) {
    constexpr int N = decltype(Nc)::value;
    r = nmax > 1 ? LineShape<T, N, 2, 2>::W : LineShape<T, N, 1, 1>::W;
  });
  return r;
}

#define IBDL_FFT2_INST(T)                                                                                       \
  template void fft2_x_r2c<T>(const T*, cplx<T>*, int, int, int, const Tw2<T>&, hipStream_t, int, const Rows2&); \
  template void fft2_x_c2r<T>(const cplx<T>*, T*, int, int, int, const Tw2<T>&, hipStream_t, int, const Rows2&); \
  template void fft2_lines<T>(cplx<T>*, int, int, const MultDesc&, const Tw2<T>&, hipStream_t, int, int64_t, int, \
                              const RowMask&);                                                                \
  template size_t fft2_table_len<T>(int, int);                                                                \
  template Tw2<T> fft2_tables<T>(int, int, const cplx<T>*, const cplx<T>*, cplx<T>*, hipStream_t);            \
  template int fft2_rows_max<T>(int);                                                                         \
  template void fft2_group_set<T>(Fft2Group&, T*, cplx<T>*, int, int, int, const Tw2<T>&);                        \
  template void fft2_groups<T>(const Fft2Group*, const Fft2Group*, int, const int2*, int, int, hipStream_t);      \
  template int fft2_lines_max<T>(int, int);
IBDL_FFT2_INST(float)
IBDL_FFT2_INST(double)

}  // namespace ibdl
