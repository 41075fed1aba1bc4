// Double-precision Krylov vector kernels (GMRES Arnoldi with classical Gram-Schmidt twice).
// Reductions are two-level with a fixed order (per-block partial sums, then one pass over the
// partials), so every dot product is deterministic.
#include <algorithm>

#include "kernels.h"

namespace ibdl {
namespace {

constexpr int kB = 256;
constexpr int kElemsPerBlock = 2048;

// partial[j * nblk + b] = sum over block b's chunk of V_j . w, for j < k
__global__ __launch_bounds__(kB) void k_multidot(const double* __restrict__ V, int64_t ldv, int k,
                                                 const double* __restrict__ w, int64_t n, int nblk,
                                                 double* __restrict__ partial) {
  __shared__ double red[kB];
  const int64_t beg = (int64_t)blockIdx.x * kElemsPerBlock;
  const int64_t end = beg + kElemsPerBlock < n ? beg + kElemsPerBlock : n;
  for (int j = 0; j < k; ++j) {
    const double* vj = V + j * ldv;
    double s = 0.0;
    for (int64_t e = beg + threadIdx.x; e < end; e += kB) s += vj[e] * w[e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = kB / 2; st > 0; st >>= 1) {
      if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
      __syncthreads();
    }
    if (threadIdx.x == 0) partial[j * nblk + blockIdx.x] = red[0];
    __syncthreads();
  }
}

__global__ void k_reduce(const double* __restrict__ partial, int nblk, double* __restrict__ out) {
  const int j = blockIdx.x;
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int b = 0; b < nblk; ++b) s += partial[j * nblk + b];
    out[j] = s;
  }
}

__global__ void k_scale(const double* __restrict__ src, double s, double* __restrict__ dst, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = src[e] * s;
}

// dst (and dst2 if set) = src / sqrt(max(*nrm2, 0)); 0 where that norm is not above floor (the
// Arnoldi breakdown, which the host detects from the same value).  Norms clamp a negative rounding
// residue to 0 but keep a NaN, so that the host sees non-finite data rather than a zero vector.
__global__ void k_scale_norm(const double* src, const double* __restrict__ nrm2, double floor, double* dst,
                             double* dst2, int64_t n) {
  const double v = *nrm2;
  const double h = sqrt(v < 0.0 ? 0.0 : v);
  const double s = (h > floor && h < INFINITY) ? 1.0 / h : 0.0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const double x = src[e] * s;
    dst[e] = x;
    if (dst2) dst2[e] = x;
  }
}

__global__ void k_axpby_d(double* __restrict__ y, double a, const double* __restrict__ x, double b, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    y[e] = a * x[e] + b * y[e];
}

// partial sums of eta * ds_i * q[i][c] over markers, per component c (ds = NULL: unit weights)
__global__ __launch_bounds__(kB) void k_border_partial(const double* __restrict__ q, const double* __restrict__ ds,
                                                       int64_t n_ib, int nq, int nblk, double* __restrict__ partial) {
  __shared__ double red[kB];
  const int c = blockIdx.y;
  const int64_t beg = (int64_t)blockIdx.x * kElemsPerBlock;
  const int64_t end = beg + kElemsPerBlock < n_ib ? beg + kElemsPerBlock : n_ib;
  double s = 0.0;
  for (int64_t i = beg + threadIdx.x; i < end; i += kB) s += (ds ? ds[i] : 1.0) * q[i * nq + c];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = kB / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[c * nblk + blockIdx.x] = red[0];
}

__global__ void k_border_final(const double* __restrict__ partial, int nblk, double eta, double* __restrict__ out) {
  const int c = blockIdx.x;
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int b = 0; b < nblk; ++b) s += partial[c * nblk + b];
    out[c] = eta * s;
  }
}

// Marker side of the transposed operator.  G holds, per marker, the interpolated adjoint grid
// fields (scalar: D_d w for d < D, then w when eta > 0; Stokes: the fields dual to A11, A12, A22
// (and eta Q1, eta Q2)); the result is
//   scalar  y_i = h^-D ds_i (sum_d n_id G_i,d - eta G_i,D) + b p_i + eta ds_i pu
//   Stokes  y_ic = h^-D ds_i sum_f (d c_f / d Q_c) G_i,f + b p_ic + eta ds_i pu_c
// with c_f the per-marker spread coefficients 2 Q1 n1, Q1 n2 + Q2 n1, 2 Q2 n2, eta Q1, eta Q2.
__global__ void k_adj_combine(int stokes, int dim, int64_t n_ib, int ng, double hDinv, double eta,
                              const double* __restrict__ G, const double* __restrict__ nrm,
                              const double* __restrict__ ds, const double* __restrict__ p, double b,
                              const double* __restrict__ pu, double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_ib) return;
  const double* Gi = G + i * ng;
  const double w = hDinv * ds[i];
  if (!stokes) {
    double s = 0.0;
    for (int d = 0; d < dim; ++d) s += nrm[i * dim + d] * Gi[d];
    if (ng > dim) s -= eta * Gi[dim];
    double v = w * s;
    if (p) v += b * p[i];
    if (pu) v += eta * ds[i] * pu[0];
    y[i] = v;
    return;
  }
  const double n1 = nrm[2 * i], n2 = nrm[2 * i + 1];
  double s1 = 2.0 * n1 * Gi[0] + n2 * Gi[1];
  double s2 = n1 * Gi[1] + 2.0 * n2 * Gi[2];
  if (ng > 3) {
    s1 += eta * Gi[3];
    s2 += eta * Gi[4];
  }
  double v1 = w * s1, v2 = w * s2;
  if (p) {
    v1 += b * p[2 * i];
    v2 += b * p[2 * i + 1];
  }
  if (pu) {
    v1 += eta * ds[i] * pu[0];
    v2 += eta * ds[i] * pu[1];
  }
  y[2 * i] = v1;
  y[2 * i + 1] = v2;
}

// Per-marker weights of the grid fields whose kernel-derivative gathers make up dL/dX:
//   scalar  [u: -mu_i] [D_d r: -h^-D ds_i Q_i n_id] [r: eta h^-D ds_i Q_i (eta > 0)]
//   Stokes  [u_c: -mu_ic] [Z_f: h^-D ds_i c_f,i for the nf spread fields]
__global__ void k_adj_coefs(int stokes, int dim, int64_t n_ib, int nc, double hDinv, double eta,
                            const double* __restrict__ mu, const double* __restrict__ q,
                            const double* __restrict__ nrm, const double* __restrict__ ds,
                            double* __restrict__ coef) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_ib) return;
  double* c = coef + i * nc;
  const double w = hDinv * ds[i];
  if (!stokes) {
    c[0] = -mu[i];
    for (int d = 0; d < dim; ++d) c[1 + d] = -w * q[i] * nrm[i * dim + d];
    if (nc > dim + 1) c[dim + 1] = eta * w * q[i];
    return;
  }
  const double q1 = q[2 * i], q2 = q[2 * i + 1], n1 = nrm[2 * i], n2 = nrm[2 * i + 1];
  c[0] = -mu[2 * i];
  c[1] = -mu[2 * i + 1];
  c[2] = w * 2.0 * q1 * n1;
  c[3] = w * (q1 * n2 + q2 * n1);
  c[4] = w * 2.0 * q2 * n2;
  if (nc > 5) {
    c[5] = w * eta * q1;
    c[6] = w * eta * q2;
  }
}

// ------------------------------------------------------------------ sums over a workgroup
// KR per-thread values at once: each wave folds them so that a lane ends with the whole wave's sum of
// one value (17 exchanges for 16 values, against 96 for a butterfly of each), then one wave adds the
// waves' sums.  The order is fixed, so the sums do not depend on scheduling, and every workgroup that
// sums the same values gets the same bits.
template <int KR> __device__ __forceinline__ double wave_fold(double (&v)[KR], int lane) {
#pragma unroll
  for (int h = KR / 2, off = 32; h >= 1; h /= 2, off /= 2) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const double a = v[i], b = v[i + h];   // (named: selecting between array elements is compiled as indexing)
      const double keep = up ? b : a, send = up ? a : b;
      v[i] = keep + __shfl_xor(send, off);
    }
  }
#pragma unroll
  for (int off = 32 / KR; off > 0; off /= 2) v[0] += __shfl_xor(v[0], off);
  return v[0];   // the sum of value lane / (64 / KR)
}

// out[0..KR) (LDS) = the workgroup's sums; part: [NT / 64][KR] of LDS.  Ends with a barrier.
template <int NT, int KR> __device__ __forceinline__ void block_fold(double (&v)[KR], double* part, double* out) {
  constexpr int NW = NT / 64, G = 64 / KR;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double s = wave_fold<KR>(v, lane);
  if (lane % G == 0) part[wave * KR + lane / G] = s;
  __syncthreads();
  if (wave == 0) {
    const int g = lane % KR, q0 = lane / KR;
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < NW; q += G)
      if (q + q0 < NW) t += part[(q + q0) * KR + g];
#pragma unroll
    for (int off = KR; off < 64; off *= 2) t += __shfl_xor(t, off);
    if (lane < KR) out[g] = t;
  }
  __syncthreads();
}

// out[j] (LDS) = the sum of p[j * nblk .. + nblk) for j < cnt, sixteen lanes per sum; ends with a barrier
__device__ __forceinline__ void sum_partials(const double* __restrict__ p, int cnt, int nblk, double* out) {
  const int l = threadIdx.x & 15;
  for (int j = threadIdx.x >> 4; j < cnt; j += kB / 16) {
    double s = 0.0;
#pragma unroll 4
    for (int b = l; b < nblk; b += 16) s += p[(int64_t)j * nblk + b];
#pragma unroll
    for (int off = 8; off > 0; off /= 2) s += __shfl_xor(s, off, 16);
    if (l == 0) out[j] = s;
  }
  __syncthreads();
}

constexpr int kArnChunk = 256;   // entries per workgroup of the blocked Arnoldi kernels, one per thread
constexpr int kArnK = 16;        // basis vectors a thread holds at a time

// ------------------------------------------------------------------ batched (segmented) vectors
// A batch vector is the concatenation of the problems' vectors; block b of a segmented dot covers
// [beg[b], end[b]) inside one problem's segment, and problem p owns blocks pb0[p] .. pb0[p+1]-1.
__global__ __launch_bounds__(kB) void k_bmultidot(const double* __restrict__ V, int64_t ldv, int k,
                                                  const double* __restrict__ w, const int64_t* __restrict__ beg,
                                                  const int64_t* __restrict__ end, int nblk,
                                                  double* __restrict__ partial) {
  __shared__ double red[kB];
  const int64_t b0 = beg[blockIdx.x], b1 = end[blockIdx.x];
  for (int j = 0; j < k; ++j) {
    const double* vj = V + j * ldv;
    double s = 0.0;
    for (int64_t e = b0 + threadIdx.x; e < b1; e += kB) s += vj[e] * w[e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = kB / 2; st > 0; st >>= 1) {
      if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
      __syncthreads();
    }
    if (threadIdx.x == 0) partial[j * nblk + blockIdx.x] = red[0];
    __syncthreads();
  }
}

// out[p * ostride + j] = sum of problem p's partial sums of dot j (grid: k x nprob)
__global__ void k_breduce(const double* __restrict__ partial, int nblk, const int* __restrict__ pb0, int ostride,
                          double* __restrict__ out) {
  const int j = blockIdx.x, p = blockIdx.y;
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int b = pb0[p]; b < pb0[p + 1]; ++b) s += partial[j * nblk + b];
    out[p * ostride + j] = s;
  }
}

// x[e] = sum_j V_j[e] Y[seg(e)][j]
__global__ void k_blincomb(const double* __restrict__ V, int64_t ldv, int k, const double* __restrict__ Y, int ys,
                           const int* __restrict__ seg, double* __restrict__ x, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const double* yp = Y + (int64_t)seg[e] * ys;
    double s = 0.0;
    for (int j = 0; j < k; ++j) s += V[j * ldv + e] * yp[j];
    x[e] = s;
  }
}

// ------------------------------------------------------------------ GMRES least squares
// The Givens-rotated Hessenberg matrix R, the rotations and the rotated right-hand side g of one
// GMRES solve live in device memory (layout gm_* below), so the least-squares problem is updated
// and solved on the device in double precision.  Step j's column is h1[i] + h2[i] (i <= j, the two
// Gram-Schmidt passes) and |w| below it; the rotations of the earlier steps are applied to it, the
// new rotation zeroes |w|, g is rotated, and res = |g[j+1]| / |b| is the Krylov residual estimate.
// Once res <= tol or the Arnoldi process breaks down the state is frozen: steps queued after that
// change nothing, and k stays the number of steps the solution uses.
__device__ __forceinline__ double* gm_cs(double* gs) { return gs + GM_HDR; }
__device__ __forceinline__ double* gm_sn(double* gs, int mx) { return gs + GM_HDR + mx; }
__device__ __forceinline__ double* gm_g(double* gs, int mx) { return gs + GM_HDR + 2 * mx; }
__device__ __forceinline__ double* gm_R(double* gs, int mx) { return gs + GM_HDR + 3 * mx + 1; }

// What a step's least-squares update reads of the state, staged in LDS when the step's kernel starts
// (beside its first vector loads) so that the update waits for no memory.
struct GivensLds {
  double c[256], s[256], col[257];
  double beta, g;   // |b|, g[j]
  int frozen;
};
__device__ __forceinline__ void givens_stage(GivensLds& G, const double* gs, int mx, int j, double bnorm2) {
  double* m = const_cast<double*>(gs);
  for (int i = threadIdx.x; i < j; i += blockDim.x) {
    G.c[i] = gm_cs(m)[i];
    G.s[i] = gm_sn(m, mx)[i];
  }
  if (threadIdx.x == 0) {
    G.frozen = j > 0 && gs[GM_DONE] != 0.0;
    G.beta = j > 0 ? gs[GM_BETA] : sqrt(bnorm2 < 0.0 ? 0.0 : bnorm2);
    G.g = j > 0 ? gm_g(m, mx)[j] : G.beta;
  }
}

// Run by one wave, after a barrier behind givens_stage (the sequential rotation sweep by lane 0).
// h1, h2: the two Gram-Schmidt passes' dots (LDS), nrm2 = |w|^2 of this step.
__device__ __forceinline__ void givens_update(GivensLds& G, const double* h1, const double* h2, double nrm2, int j, int mx,
                                              double tol, double* gs) {
  const int lane = threadIdx.x & 63;
  if (G.frozen) return;
  for (int i = lane; i <= j; i += 64) G.col[i] = h1[i] + h2[i];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) {
    double* g = gm_g(gs, mx);
    const double beta = G.beta, hn = sqrt(nrm2 < 0.0 ? 0.0 : nrm2);
    if (j == 0) {
      gs[GM_BETA] = beta;
      g[0] = beta;
    }
    double cur = G.col[0];
#pragma unroll 4
    for (int i = 0; i < j; ++i) {
      const double nxt = G.col[i + 1], c = G.c[i], sv = G.s[i];
      G.col[i] = c * cur + sv * nxt;
      cur = -sv * cur + c * nxt;
    }
    G.col[j] = cur;
    double res = 0.0;
    bool stop = true;
    if (beta > 0.0) {
      const double r = hypot(cur, hn);
      const double c = cur / r, sv = hn / r;
      gm_cs(gs)[j] = c;
      gm_sn(gs, mx)[j] = sv;
      G.col[j] = r;
      const double gn = -sv * G.g;
      g[j + 1] = gn;
      g[j] = c * G.g;
      res = fabs(gn) / beta;
      const bool breakdown = !(hn > 1e-300 * beta);
      stop = res <= tol || breakdown || !(res == res);
      gs[GM_K] = (double)(j + 1);
    } else {
      gs[GM_K] = 0.0;
    }
    gs[GM_RES] = res;
    gs[GM_HN] = hn;
    gs[GM_DONE] = stop ? 1.0 : 0.0;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  double* R = gm_R(gs, mx) + (int64_t)j * (mx + 1);
  for (int i = lane; i <= j; i += 64) R[i] = G.col[i];
}

// By the wave that ran givens_update: the state's record to host-mapped memory (gm_record.h)
__device__ __forceinline__ void publish_state(const double* gs, double* dst, unsigned seq) {
  __threadfence_block();
  const int lane = threadIdx.x & 63;
  unsigned long long w = 0;
  if (lane < GM_PUB) {
    const double v = *const_cast<const volatile double*>(gs + lane);
    w = __builtin_bit_cast(unsigned long long, v);
  }
  unsigned long long c = lane < GM_PUB ? gm_pub_mix(w, lane) : 0;
#pragma unroll
  for (int off = 1; off < 8; off *= 2) c ^= __shfl_xor(c, off);
  if (lane == GM_PUB) w = c ^ gm_pub_key(seq);
  if (lane <= GM_PUB)
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(dst) + lane, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------------------ blocked Arnoldi step
// Three launches over 256-entry blocks, one entry per thread, sixteen basis vectors in registers at a
// time: their loads are issued first and serve the update and the dots.
//   k_arn0  pout[j][b] = block b's part of V_j . w
//   k_arn1  h1 = sums of pin (reduced in every workgroup, in the same order), w -= V h1,
//           pout[j][b] = parts of V_j . w (j < k) and of w . w (j = k)
//   k_arn2  h2 likewise, |w|^2 (arn_norm2), V_k (and vdst2) = (w - V h2) / |w|; workgroup 0 runs the
//           least-squares update and publishes the state.  w itself stays as k_arn1 left it.
// What bounds a step at these lengths is the chain of each launch (read what the last launch wrote,
// fold, write; a vector is a few tens of KB), so it has one launch and two folds fewer than with an LDS
// tree per eight dots and a norm pass of its own: 20.4 -> 13.6 us a step at 4,096 unknowns (10 basis
// vectors), 24 -> 14.5 at 2,050, 21 -> 15 at 18,492.
__device__ __forceinline__ void arn_load(double (&v)[kArnK], const double* __restrict__ V, int64_t ldv, int c0, int k,
                                         int64_t e, bool in) {
  // (unconditional loads at clamped places, so that no branch stands between them)
  const double* p = V + (in ? e : 0);
#pragma unroll
  for (int g = 0; g < kArnK; ++g) v[g] = p[(int64_t)(c0 + g < k ? c0 + g : k - 1) * ldv];
#pragma unroll
  for (int g = 0; g < kArnK; ++g) v[g] = in && c0 + g < k ? v[g] : 0.0;
}

__global__ __launch_bounds__(kB) void k_arn0(const double* __restrict__ V, int64_t ldv, int k,
                                             const double* __restrict__ w, int64_t n, int nblk,
                                             double* __restrict__ pout) {
  __shared__ double part[kB / 64 * kArnK], out[kArnK];
  const int64_t e = (int64_t)blockIdx.x * kArnChunk + threadIdx.x;
  const bool in = e < n;
  const double we = in ? w[e] : 0.0;
  for (int c0 = 0; c0 < k; c0 += kArnK) {
    double v[kArnK];
    arn_load(v, V, ldv, c0, k, e, in);
#pragma unroll
    for (int g = 0; g < kArnK; ++g) v[g] *= we;
    block_fold<kB, kArnK>(v, part, out);
    if (threadIdx.x < kArnK && c0 + (int)threadIdx.x < k) pout[(int64_t)(c0 + threadIdx.x) * nblk + blockIdx.x] = out[threadIdx.x];
  }
}

__global__ __launch_bounds__(kB) void k_arn1(const double* __restrict__ V, int64_t ldv, int k, double* __restrict__ w,
                                             int64_t n, int nblk, const double* __restrict__ pin,
                                             double* __restrict__ hout, double* __restrict__ pout) {
  __shared__ double part[kB / 64 * kArnK], out[kArnK], hs[256 + kArnK];
  const int64_t e = (int64_t)blockIdx.x * kArnChunk + threadIdx.x;
  const bool in = e < n;
  double we = in ? w[e] : 0.0;
  double v[kArnK];
  arn_load(v, V, ldv, 0, k, e, in);
  sum_partials(pin, k, nblk, hs);
  if (threadIdx.x < kArnK) hs[k + threadIdx.x] = 0.0;
  if (blockIdx.x == 0)
    for (int j = threadIdx.x; j < k; j += kB) hout[j] = hs[j];
  __syncthreads();
  for (int c0 = 0; c0 < k; c0 += kArnK) {
    if (c0 > 0) arn_load(v, V, ldv, c0, k, e, in);
#pragma unroll
    for (int g = 0; g < kArnK; ++g) we -= v[g] * hs[c0 + g];
  }
  if (in) w[e] = we;
  for (int c0 = 0; c0 <= k; c0 += kArnK) {   // k dots, then w . w
    if (k > kArnK) arn_load(v, V, ldv, c0, k, e, in);
    double d[kArnK];
#pragma unroll
    for (int g = 0; g < kArnK; ++g) d[g] = (c0 + g == k ? we : (c0 + g < k ? v[g] : 0.0)) * we;
    block_fold<kB, kArnK>(d, part, out);
    if (threadIdx.x < kArnK && c0 + (int)threadIdx.x <= k) pout[(int64_t)(c0 + threadIdx.x) * nblk + blockIdx.x] = out[threadIdx.x];
  }
}

// |w - V h|^2, h = V . w (hs[0..k), and w . w at hs[k]), for an orthonormal V: the update takes the h
// components out of w, so this is w . w - |h|^2, and the rounding of that difference stays below a few
// units in its last place while it is more than half of w . w.  h is what the first pass's rounding left
// behind, so it always is unless w is at the level of that rounding itself (an invariant Krylov space).
// There the difference holds no digits and may come out negative, and every workgroup sums the updated
// entries instead: all n of them, in the same order, so that all have the same bits (w = 0 needs no sum).
__device__ __forceinline__ double arn_norm2(const double* __restrict__ V, int64_t ldv, int k, const double* __restrict__ w,
                                            int64_t n, const double* hs, double* red) {
  double nrm2 = hs[k];
  for (int j = 0; j < k; ++j) nrm2 -= hs[j] * hs[j];
  if (!(nrm2 <= 0.5 * hs[k]) || hs[k] == 0.0) return nrm2;
  double s = 0.0;
  for (int64_t e = threadIdx.x; e < n; e += kB) {
    double x = w[e];
    for (int j = 0; j < k; ++j) x -= V[(int64_t)j * ldv + e] * hs[j];
    s += x * x;
  }
#pragma unroll
  for (int off = 32; off > 0; off /= 2) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ __launch_bounds__(kB) void k_arn2(const double* __restrict__ V, int64_t ldv, int k,
                                             const double* __restrict__ w, int64_t n, int nblk,
                                             const double* __restrict__ pin, const double* __restrict__ h1g,
                                             const double* __restrict__ bn2, double* gs, int mx, double tol, double* dst,
                                             unsigned seq, double* __restrict__ vdst, double* __restrict__ vdst2) {
  __shared__ double hs[256 + kArnK], h1[256], red[kB / 64];
  __shared__ GivensLds G;
  const int64_t e = (int64_t)blockIdx.x * kArnChunk + threadIdx.x;
  const bool in = e < n;
  double we = in ? w[e] : 0.0;
  double v[kArnK];
  arn_load(v, V, ldv, 0, k, e, in);
  if (blockIdx.x == 0) {
    givens_stage(G, gs, mx, k - 1, *bn2);
    for (int j = threadIdx.x; j < k; j += kB) h1[j] = h1g[j];
  }
  sum_partials(pin, k + 1, nblk, hs);
  const double nrm2 = arn_norm2(V, ldv, k, w, n, hs, red);
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    givens_update(G, h1, hs, nrm2, k - 1, mx, tol, gs);
    publish_state(gs, dst, seq);
  }
  for (int c0 = 0; c0 < k; c0 += kArnK) {
    if (c0 > 0) arn_load(v, V, ldv, c0, k, e, in);
#pragma unroll
    for (int g = 0; g < kArnK; ++g)
      if (c0 + g < k) we -= v[g] * hs[c0 + g];
  }
  const double hn = sqrt(nrm2 < 0.0 ? 0.0 : nrm2);
  const double sc = (hn > 0.0 && hn < INFINITY) ? 1.0 / hn : 0.0;
  if (in) {
    const double x = we * sc;
    vdst[e] = x;
    if (vdst2) vdst2[e] = x;
  }
}

// ------------------------------------------------------------------ Arnoldi step by one workgroup
// Both Gram-Schmidt passes, |w|, the least-squares update and the normalisation, for vectors of at
// most NT R entries: thread t holds entries t + r NT of w and of KR basis vectors at a time in
// registers (read once per step while k <= KR).  Returns false (and writes nothing) where the state
// is frozen and SKIP is set.
template <int NT, int R, int KR, bool SKIP>
__device__ __forceinline__ bool arnoldi_wg(const double* __restrict__ V, int64_t ldv, int k, const double* w, int64_t n,
                                           double bnorm2, double* gs, int mx, double tol, double* vdst, double* vdst2,
                                           double floor_rel) {
  __shared__ double part[NT / 64 * KR], hv[2][256 + KR], red[NT / 64];
  __shared__ GivensLds G;
  double we[R], v[KR][R];
  auto load = [&](int c0) {
#pragma unroll
    for (int r = 0; r < R; ++r) {   // (unconditional loads at clamped places, so that no branch stands between them)
      const int64_t e = threadIdx.x + (int64_t)r * NT;
      const double* p = V + (e < n ? e : 0);
#pragma unroll
      for (int g = 0; g < KR; ++g) v[g][r] = p[(int64_t)(c0 + g < k ? c0 + g : k - 1) * ldv];
#pragma unroll
      for (int g = 0; g < KR; ++g) v[g][r] = c0 + g < k && e < n ? v[g][r] : 0.0;
    }
  };
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t e = threadIdx.x + (int64_t)r * NT;
    we[r] = e < n ? w[e] : 0.0;
  }
  load(0);
  givens_stage(G, gs, mx, k - 1, bnorm2);
  __syncthreads();
  if (SKIP && G.frozen) return false;
  for (int pass = 0; pass < 2; ++pass) {
    for (int c0 = 0; c0 < k; c0 += KR) {
      if (c0 > 0 || (pass > 0 && k > KR)) load(c0);
      double d[KR];
#pragma unroll
      for (int g = 0; g < KR; ++g) {
        d[g] = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) d[g] += v[g][r] * we[r];
      }
      block_fold<NT, KR>(d, part, hv[pass] + c0);
    }
    for (int c0 = 0; c0 < k; c0 += KR) {
      if (k > KR) load(c0);
#pragma unroll
      for (int g = 0; g < KR; ++g) {
        const double h = hv[pass][c0 + g];
#pragma unroll
        for (int r = 0; r < R; ++r) we[r] -= v[g][r] * h;
      }
    }
  }
  double sq = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) sq += we[r] * we[r];
#pragma unroll
  for (int off = 32; off > 0; off /= 2) sq += __shfl_xor(sq, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
  __syncthreads();
  double nrm2 = 0.0;
#pragma unroll
  for (int q = 0; q < NT / 64; ++q) nrm2 += red[q];
  if (threadIdx.x < 64) givens_update(G, hv[0], hv[1], nrm2, k - 1, mx, tol, gs);
  const double hn = sqrt(nrm2 < 0.0 ? 0.0 : nrm2);
  const double sc = (hn > floor_rel * G.beta && hn < INFINITY) ? 1.0 / hn : 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t e = threadIdx.x + (int64_t)r * NT;
    if (e < n) {
      const double x = we[r] * sc;
      vdst[e] = x;
      if (vdst2) vdst2[e] = x;
    }
  }
  return true;
}

template <int NT, int R, int KR>
__global__ __launch_bounds__(NT) void k_arnoldi_one(const double* __restrict__ V, int64_t ldv, int k, const double* w,
                                                    int64_t n, const double* __restrict__ bn2, double* gs, int mx,
                                                    double tol, double* dst, unsigned seq, double* vdst, double* vdst2) {
  arnoldi_wg<NT, R, KR, false>(V, ldv, k, w, n, *bn2, gs, mx, tol, vdst, vdst2, 0.0);
  if (threadIdx.x < 64) publish_state(gs, dst, seq);
}

// ------------------------------------------------------------------ start, finish, residual
// |b|^2 and v0 (and v02) = b / |b| (0 where |b| is 0 or not finite), one workgroup, n <= 16 * 1024
constexpr int kOneWg = 16 * 1024;
__global__ __launch_bounds__(1024) void k_start_one(const double* __restrict__ b, int64_t n, double* bn2, double* v0,
                                                    double* v02) {
  __shared__ double red[16];
  double x[16], s = 0.0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t e = threadIdx.x + (int64_t)r * 1024;
    x[r] = e < n ? b[e] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) s += x[r] * x[r];
#pragma unroll
  for (int off = 32; off > 0; off /= 2) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  double v = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) v += red[q];
  if (threadIdx.x == 0) *bn2 = v;
  const double h = sqrt(v < 0.0 ? 0.0 : v);
  const double sc = (h > 0.0 && h < INFINITY) ? 1.0 / h : 0.0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t e = threadIdx.x + (int64_t)r * 1024;
    if (e < n) {
      v0[e] = x[r] * sc;
      if (v02) v02[e] = x[r] * sc;
    }
  }
}

// partial[b] = block b's part of |b - a|^2
__global__ __launch_bounds__(kB) void k_resid_partial(const double* __restrict__ b, const double* __restrict__ a,
                                                      int64_t n, double* __restrict__ partial) {
  __shared__ double red[kB / 64];
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < kElemsPerBlock / kB; ++r) {
    const int64_t e = (int64_t)blockIdx.x * kElemsPerBlock + r * kB + threadIdx.x;
    const double d = e < n ? b[e] - a[e] : 0.0;
    s += d * d;
  }
#pragma unroll
  for (int off = 32; off > 0; off /= 2) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// x = V y with y = R^-1 g of the k = gs[GM_K] steps: every workgroup solves the triangle itself (k <= 64:
// by its first wave, lane i holding g_i, from LDS; longer ones column by column) and forms its part of x.
// gate: nothing unless the state's convergence flag is set (a finish queued behind a step that the
// host predicts to be the last, before it has seen that step's result).
__global__ __launch_bounds__(kB) void k_gmres_finish(const double* __restrict__ V, int64_t ldv, const double* gs, int mx,
                                                     double* __restrict__ x, int64_t n, int gate) {
  __shared__ double tri[64 * 64];
  __shared__ double ys[256];
  if (gate && gs[GM_DONE] == 0.0) return;
  const int k = (int)gs[GM_K];
  double* m = const_cast<double*>(gs);
  const double* R = gm_R(m, mx);
  const double* g = gm_g(m, mx);
  if (k <= 64) {
    for (int q = threadIdx.x; q < k * k; q += kB) {
      const int c = q / k, i = q - c * k;
      tri[c * 64 + i] = i <= c ? R[(int64_t)c * (mx + 1) + i] : 0.0;
    }
    double gi = (int)threadIdx.x < k ? g[threadIdx.x] : 0.0;
    __syncthreads();
    if (threadIdx.x < 64) {
      for (int c = k - 1; c >= 0; --c) {
        const double y = __shfl(gi, c) / tri[c * 64 + c];
        if ((int)threadIdx.x == c) ys[c] = y;
        else if ((int)threadIdx.x < c) gi -= tri[c * 64 + threadIdx.x] * y;
      }
    }
    __syncthreads();
  } else {
    for (int i = threadIdx.x; i < k; i += kB) ys[i] = g[i];
    __syncthreads();
    for (int c = k - 1; c >= 0; --c) {
      const double* rc = R + (int64_t)c * (mx + 1);
      const double y = ys[c] / rc[c];
      __syncthreads();
      for (int i = threadIdx.x; i <= c; i += kB) ys[i] = i == c ? y : ys[i] - rc[i] * y;
      __syncthreads();
    }
  }
  for (int64_t e = (int64_t)blockIdx.x * kB + threadIdx.x; e < n; e += (int64_t)gridDim.x * kB) {
    double s = 0.0;
#pragma unroll 8
    for (int j = 0; j < k; ++j) s += V[j * ldv + e] * ys[j];
    x[e] = s;
  }
}

// ------------------------------------------------------------------ batched GMRES on the device
// One workgroup per problem does a whole Arnoldi step of its problem on its segment
// [off[p], off[p] + len[p]) of the batch vectors and its own state gs + p * gstride.  A problem whose
// state was already frozen writes zeros there (its later applies run on zeros) and changes nothing
// else.  The step number j comes from the host.
template <int NT, int R, int KR>
__global__ __launch_bounds__(NT) void k_batch_arnoldi_wg(const double* __restrict__ V, int64_t ldv, int j,
                                                         const double* __restrict__ w, const int64_t* __restrict__ off,
                                                         const int64_t* __restrict__ len,
                                                         const double* __restrict__ bn2, double* gsb, int64_t gstride,
                                                         int mx, double tol, double* __restrict__ vnext,
                                                         double* __restrict__ xin, double* dst, unsigned seq) {
  const int p = blockIdx.x;
  const int64_t beg = off[p], n = len[p];
  double* gs = gsb + (int64_t)p * gstride;
  const bool ran = arnoldi_wg<NT, R, KR, true>(V + beg, ldv, j + 1, w + beg, n, bn2[p], gs, mx, tol, vnext + beg,
                                               xin ? xin + beg : nullptr, 1e-300);
  if (threadIdx.x < 64) publish_state(gs, dst + (int64_t)p * GM_REC, seq);
  if (ran) return;
  for (int64_t e = threadIdx.x; e < n; e += NT) {
    vnext[beg + e] = 0.0;
    if (xin) xin[beg + e] = 0.0;
  }
}

// The same for problems of any length, w in memory
__global__ __launch_bounds__(kB) void k_batch_arnoldi(const double* __restrict__ V, int64_t ldv, int j,
                                                      double* __restrict__ w, const int64_t* __restrict__ off,
                                                      const int64_t* __restrict__ len, const double* __restrict__ bn2,
                                                      double* gsb, int64_t gstride, int mx, double tol,
                                                      double* __restrict__ vnext, double* __restrict__ xin, double* dst,
                                                      unsigned seq) {
  __shared__ double part[kB / 64 * kArnK], hv[2][256 + kArnK], out[kArnK];
  __shared__ GivensLds G;
  const int p = blockIdx.x;
  const int64_t beg = off[p], n = len[p];
  double* gs = gsb + (int64_t)p * gstride;
  givens_stage(G, gs, mx, j, bn2[p]);
  __syncthreads();
  if (G.frozen) {
    if (threadIdx.x < 64) publish_state(gs, dst + (int64_t)p * GM_REC, seq);
    for (int64_t e = threadIdx.x; e < n; e += kB) {
      vnext[beg + e] = 0.0;
      if (xin) xin[beg + e] = 0.0;
    }
    return;
  }
  const int k = j + 1;
  double* wp = w + beg;
  const double* Vp = V + beg;
  double nrm2 = 0.0;
  for (int pass = 0; pass < 2; ++pass) {
    for (int c0 = 0; c0 < k; c0 += kArnK) {
      double d[kArnK];
#pragma unroll
      for (int g = 0; g < kArnK; ++g) d[g] = 0.0;
      for (int64_t e = threadIdx.x; e < n; e += kB) {
        const double we = wp[e];
        double v[kArnK];
        arn_load(v, Vp, ldv, c0, k, e, true);
#pragma unroll
        for (int g = 0; g < kArnK; ++g) d[g] += v[g] * we;
      }
      block_fold<kB, kArnK>(d, part, hv[pass] + c0);
    }
    double sq[kArnK];
#pragma unroll
    for (int g = 0; g < kArnK; ++g) sq[g] = 0.0;
    for (int64_t e = threadIdx.x; e < n; e += kB) {
      double we = wp[e];
      for (int i = 0; i < k; ++i) we -= Vp[(int64_t)i * ldv + e] * hv[pass][i];
      wp[e] = we;
      sq[0] += we * we;
    }
    __syncthreads();
    if (pass == 1) {
      block_fold<kB, kArnK>(sq, part, out);
      nrm2 = out[0];
    }
  }
  if (threadIdx.x < 64) {
    givens_update(G, hv[0], hv[1], nrm2, j, mx, tol, gs);
    publish_state(gs, dst + (int64_t)p * GM_REC, seq);
  }
  const double hn = sqrt(nrm2 < 0.0 ? 0.0 : nrm2);
  const double sc = (hn > 1e-300 * G.beta && hn < INFINITY) ? 1.0 / hn : 0.0;
  for (int64_t e = threadIdx.x; e < n; e += kB) {
    const double x = wp[e] * sc;
    vnext[beg + e] = x;
    if (xin) xin[beg + e] = x;
  }
}

// Problem p's segment of a batch vector to or from its own array: to_batch: base[off[p] + e] =
// ptr[p][e]; otherwise ptr[p][e] = base[off[p] + e] (one launch for every problem).
__global__ void k_seg_copy(const double* const* __restrict__ ptr, const int64_t* __restrict__ off,
                           const int64_t* __restrict__ len, double* __restrict__ base, int to_batch) {
  const int p = blockIdx.y;
  const int64_t n = len[p];
  double* seg = base + off[p];
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    if (to_batch) seg[e] = ptr[p][e];
    else const_cast<double*>(ptr[p])[e] = seg[e];
  }
}

// V[0] segment of problem p = b / |b| (0 when |b| is 0 or not finite), also into xin
__global__ void k_batch_start(const double* __restrict__ b, const int64_t* __restrict__ off,
                              const int64_t* __restrict__ len, const double* __restrict__ bn2,
                              double* __restrict__ v0, double* __restrict__ xin) {
  const int p = blockIdx.x;
  const double nb = sqrt(bn2[p] < 0.0 ? 0.0 : bn2[p]);
  const double sc = (nb > 0.0 && nb < INFINITY) ? 1.0 / nb : 0.0;
  for (int64_t e = threadIdx.x; e < len[p]; e += blockDim.x) {
    const double x = b[off[p] + e] * sc;
    v0[off[p] + e] = x;
    if (xin) xin[off[p] + e] = x;
  }
}

// Per problem: y = R^-1 g of its GM_K steps into Y[p][0..kmax) (zeros beyond its own count)
__global__ __launch_bounds__(kB) void k_batch_y(double* gsb, int64_t gstride, int mx, int kmax, double* Y, int ys) {
  __shared__ double gv[256];
  __shared__ double yv;
  double* gs = gsb + (int64_t)blockIdx.x * gstride;
  const int k = (int)gs[GM_K];
  const double* R = gm_R(gs, mx);
  const double* g = gm_g(gs, mx);
  double* y = Y + (int64_t)blockIdx.x * ys;
  for (int i = threadIdx.x; i < k; i += kB) gv[i] = g[i];
  for (int i = k + threadIdx.x; i < kmax; i += kB) y[i] = 0.0;
  __syncthreads();
  for (int c = k - 1; c >= 0; --c) {
    const double* rc = R + (int64_t)c * (mx + 1);
    if (threadIdx.x == 0) {
      yv = gv[c] / rc[c];
      y[c] = yv;
    }
    __syncthreads();
    const double v = yv;
    for (int i = threadIdx.x; i < c; i += kB) gv[i] -= rc[i] * v;
    __syncthreads();
  }
}

inline unsigned blocks_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (unsigned)(b > 4096 ? 4096 : (b < 1 ? 1 : b));
}

}  // namespace

size_t kr_gmres_state_doubles(int mx) { return (size_t)GM_HDR + 3 * (size_t)mx + 1 + (size_t)mx * (mx + 1); }

void kr_gmres_finish(const double* gs, int mx, const double* V, int64_t ldv, double* x, int64_t n, bool gate,
                     hipStream_t st) {
  if (mx > 256) throw Error(-1, "kr_gmres_finish: at most 256 basis vectors");
  hipLaunchKernelGGL(k_gmres_finish, dim3(blocks_for(n)), dim3(kB), 0, st, V, ldv, gs, mx, x, n, gate ? 1 : 0);
  IBDL_LAUNCH_CHECK();
}

void kr_gmres_start(const double* b, int64_t n, double* partial, int nblk, double* bn2, double* v0, double* v02,
                    hipStream_t st) {
  if (n <= kOneWg) {
    hipLaunchKernelGGL(k_start_one, dim3(1), dim3(1024), 0, st, b, n, bn2, v0, v02);
    IBDL_LAUNCH_CHECK();
    return;
  }
  kr_multidot(b, n, 1, b, n, partial, nblk, bn2, st);
  kr_scale_norm(b, bn2, 0.0, v0, v02, n, st);
}

void kr_resid_norm2(const double* b, const double* a, int64_t n, double* partial, int nblk, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_resid_partial, dim3(nblk), dim3(kB), 0, st, b, a, n, partial);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(64), 0, st, partial, nblk, out);
  IBDL_LAUNCH_CHECK();
}

int kr_nblk(int64_t n) { return (int)((n + kElemsPerBlock - 1) / kElemsPerBlock) > 0 ? (int)((n + kElemsPerBlock - 1) / kElemsPerBlock) : 1; }

void kr_multidot(const double* V, int64_t ldv, int k, const double* w, int64_t n, double* partial, int nblk,
                 double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_multidot, dim3(nblk), dim3(kB), 0, st, V, ldv, k, w, n, nblk, partial);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_reduce, dim3(k), dim3(64), 0, st, partial, nblk, out);
  IBDL_LAUNCH_CHECK();
}

void kr_scale(const double* src, double s, double* dst, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_scale, dim3(blocks_for(n)), dim3(256), 0, st, src, s, dst, n);
  IBDL_LAUNCH_CHECK();
}

void kr_scale_norm(const double* src, const double* nrm2, double floor, double* dst, double* dst2, int64_t n,
                   hipStream_t st) {
  hipLaunchKernelGGL(k_scale_norm, dim3(blocks_for(n)), dim3(256), 0, st, src, nrm2, floor, dst, dst2, n);
  IBDL_LAUNCH_CHECK();
}

void kr_axpby(double* y, double a, const double* x, double b, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_axpby_d, dim3(blocks_for(n)), dim3(256), 0, st, y, a, x, b, n);
  IBDL_LAUNCH_CHECK();
}

void kr_border(const double* q, const double* ds, int64_t n_ib, int nq, double eta, double* out, double* partial,
               int nblk, hipStream_t st) {
  hipLaunchKernelGGL(k_border_partial, dim3(nblk, nq), dim3(kB), 0, st, q, ds, n_ib, nq, nblk, partial);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_border_final, dim3(nq), dim3(64), 0, st, partial, nblk, eta, out);
  IBDL_LAUNCH_CHECK();
}

int kr_arnoldi_nblk(int64_t n) { return (int)((n + kArnChunk - 1) / kArnChunk) > 0 ? (int)((n + kArnChunk - 1) / kArnChunk) : 1; }

void kr_arnoldi_step(const double* V, int64_t ldv, int k, double* w, int64_t n, double* partial, int nblk, double* h,
                     double* gs, int mx, double tol, double* host_dst, unsigned seq, double* vdst, double* vdst2,
                     hipStream_t st) {
  if (k < 1 || k > mx || mx > 256) throw Error(-2, "Arnoldi step: 1 <= k <= mx <= 256");
  if (w == vdst || w == vdst2) throw Error(-2, "Arnoldi step: w must not be one of its outputs");
  const double* bn2 = h + GM_BNORM2_AT;
  // One workgroup while two entries per thread hold the vectors (9.4 us a step at 269 unknowns, 13.6 for
  // the three launches); beyond that the basis vectors' reads want more than one CU.
  if (n <= 256)
    hipLaunchKernelGGL((k_arnoldi_one<256, 1, 16>), dim3(1), dim3(256), 0, st, V, ldv, k, w, n, bn2, gs, mx, tol, host_dst,
                       seq, vdst, vdst2);
  else if (n <= kArnoldiOne)
    hipLaunchKernelGGL((k_arnoldi_one<512, 2, 16>), dim3(1), dim3(512), 0, st, V, ldv, k, w, n, bn2, gs, mx, tol,
                       host_dst, seq, vdst, vdst2);
  else {
    double* p0 = partial;
    double* p1 = partial + (int64_t)k * nblk;
    hipLaunchKernelGGL(k_arn0, dim3(nblk), dim3(kB), 0, st, V, ldv, k, w, n, nblk, p0);
    IBDL_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_arn1, dim3(nblk), dim3(kB), 0, st, V, ldv, k, w, n, nblk, p0, h, p1);
    IBDL_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_arn2, dim3(nblk), dim3(kB), 0, st, V, ldv, k, w, n, nblk, p1, h, bn2, gs, mx, tol, host_dst,
                       seq, vdst, vdst2);
  }
  IBDL_LAUNCH_CHECK();
}

void kb_multidot(const double* V, int64_t ldv, int k, const double* w, const KrylovSegments& sg, double* partial,
                 int ostride, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_bmultidot, dim3(sg.nblk), dim3(kB), 0, st, V, ldv, k, w, sg.beg, sg.end, sg.nblk, partial);
  IBDL_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_breduce, dim3(k, sg.nprob), dim3(64), 0, st, partial, sg.nblk, sg.pb0, ostride, out);
  IBDL_LAUNCH_CHECK();
}

void kb_lincomb(const double* V, int64_t ldv, int k, const double* Y, int ys, const KrylovSegments& sg, double* x,
                hipStream_t st) {
  hipLaunchKernelGGL(k_blincomb, dim3(blocks_for(sg.n)), dim3(256), 0, st, V, ldv, k, Y, ys, sg.seg, x, sg.n);
  IBDL_LAUNCH_CHECK();
}

void kb_seg_copy(const double* const* ptr, const int64_t* off, const int64_t* len, int np, int64_t maxlen,
                 double* base, bool to_batch, hipStream_t st) {
  const unsigned bx = (unsigned)std::min<int64_t>((maxlen + 255) / 256, 64);
  hipLaunchKernelGGL(k_seg_copy, dim3(bx > 0 ? bx : 1, np), dim3(256), 0, st, ptr, off, len, base, to_batch ? 1 : 0);
  IBDL_LAUNCH_CHECK();
}

void kb_gmres_start(const double* b, const int64_t* off, const int64_t* len, int np, const double* bn2, double* v0,
                    double* xin, hipStream_t st) {
  hipLaunchKernelGGL(k_batch_start, dim3(np), dim3(256), 0, st, b, off, len, bn2, v0, xin);
  IBDL_LAUNCH_CHECK();
}

void kb_arnoldi(const double* V, int64_t ldv, int j, double* w, const int64_t* off, const int64_t* len, int np,
                int64_t maxlen, const double* bn2, double* gsb, int64_t gstride, int mx, double tol, double* vnext,
                double* xin, double* host_dst, unsigned seq, hipStream_t st) {
  if (j < 0 || j >= mx || mx > 256) throw Error(-2, "kb_arnoldi: 0 <= j < mx <= 256");
  auto wg = [&](auto tc, auto rc, auto kc) {
    constexpr int NT = decltype(tc)::value;
    hipLaunchKernelGGL((k_batch_arnoldi_wg<NT, decltype(rc)::value, decltype(kc)::value>), dim3(np), dim3(NT), 0, st, V,
                       ldv, j, w, off, len, bn2, gsb, gstride, mx, tol, vnext, xin, host_dst, seq);
  };
  using std::integral_constant;
  if (maxlen <= 1024) wg(integral_constant<int, 512>{}, integral_constant<int, 2>{}, integral_constant<int, 16>{});
  else if (maxlen <= 2048) wg(integral_constant<int, 1024>{}, integral_constant<int, 2>{}, integral_constant<int, 8>{});
  else if (maxlen <= 4096) wg(integral_constant<int, 1024>{}, integral_constant<int, 4>{}, integral_constant<int, 4>{});
  else
    hipLaunchKernelGGL(k_batch_arnoldi, dim3(np), dim3(kB), 0, st, V, ldv, j, w, off, len, bn2, gsb, gstride, mx, tol,
                       vnext, xin, host_dst, seq);
  IBDL_LAUNCH_CHECK();
}

void kb_gmres_y(double* gsb, int64_t gstride, int np, int mx, int kmax, double* Y, int ys, hipStream_t st) {
  hipLaunchKernelGGL(k_batch_y, dim3(np), dim3(kB), 0, st, gsb, gstride, mx, kmax, Y, ys);
  IBDL_LAUNCH_CHECK();
}

void adj_combine(int stokes, int dim, int64_t n_ib, int ng, double hDinv, double eta, const double* G,
                 const double* nrm, const double* ds, const double* p, double b, const double* pu, double* y,
                 hipStream_t st) {
  hipLaunchKernelGGL(k_adj_combine, dim3((unsigned)((n_ib + 255) / 256)), dim3(256), 0, st, stokes, dim, n_ib, ng,
                     hDinv, eta, G, nrm, ds, p, b, pu, y);
  IBDL_LAUNCH_CHECK();
}

void adj_coefs(int stokes, int dim, int64_t n_ib, int nc, double hDinv, double eta, const double* mu,
               const double* q, const double* nrm, const double* ds, double* coef, hipStream_t st) {
  hipLaunchKernelGGL(k_adj_coefs, dim3((unsigned)((n_ib + 255) / 256)), dim3(256), 0, st, stokes, dim, n_ib, nc,
                     hDinv, eta, mu, q, nrm, ds, coef);
  IBDL_LAUNCH_CHECK();
}

}  // namespace ibdl
