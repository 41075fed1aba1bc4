// The record that a GMRES step publishes to the host: GM_PUB scalars of the least-squares state (see
// kr_gmres_state_doubles) and a check word.
//
// The device stores the words without a fence, so the host may find some of an earlier step's (or of
// zeroed memory) among them, and takes the record once the check word fits: the exclusive or of a key made
// of the step's sequence number and of every word, mixed with its place.  Unmixed, equal changes in two
// stale words would cancel (GM_K and GM_DONE both go from 0.0 to 1.0 in a first step that solves).  Mixed,
// the check is a 64-bit hash: a mixed-up record passes with a probability of about 2^-64.
#pragma once

namespace ibdl {

enum { GM_BETA = 0, GM_RES = 1, GM_K = 2, GM_DONE = 3, GM_HN = 4, GM_PUB = 5, GM_HDR = 16 };
constexpr int GM_REC = 8;   // doubles per record (64 bytes)

__host__ __device__ inline unsigned long long gm_pub_key(unsigned seq) { return (seq + 1ull) * 0x9E3779B97F4A7C15ull; }

// word i of the record as it enters the check word: its halves combined (small integers held in double
// precision have no low bits), times an odd number of its own
__host__ __device__ inline unsigned long long gm_pub_mix(unsigned long long w, int i) {
  w = (w ^ (w >> 32)) * (0xBF58476D1CE4E5B9ull * (2ull * (unsigned)i + 1ull));
  return w ^ (w >> 29);
}

// whether rec holds the record of step number seq; its scalars to out
inline bool gm_pub_read(const volatile double* rec, unsigned seq, double* out) {
  unsigned long long c = gm_pub_key(seq), w;
  for (int i = 0; i <= GM_PUB; ++i) {
    const double v = rec[i];
    __builtin_memcpy(&w, &v, 8);
    c ^= i < GM_PUB ? gm_pub_mix(w, i) : w;
    if (i < GM_PUB) out[i] = v;
  }
  return c == 0;
}

}  // namespace ibdl
