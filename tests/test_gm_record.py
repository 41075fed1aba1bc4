"""The record a GMRES step publishes (gm_record.h), on the CPU: a record is taken when every word is its
step's, and never when some are an earlier record's or zeros, whichever words they are.  The scalars run
over what the steps of solves publish, with the pairs of equal changes among them: GM_K and GM_DONE both 0 to
1, 1 to 0, or one each way, and residual, |b| and |w| that change by the same bits."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_07403_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include <vector>
#include "gm_record.h"
using namespace ibdl;

struct Rec { double v[GM_REC]; unsigned seq; };

static Rec make(double beta, double res, double k, double done, double hn, unsigned seq) {
  Rec r{};
  r.seq = seq;
  r.v[GM_BETA] = beta; r.v[GM_RES] = res; r.v[GM_K] = k; r.v[GM_DONE] = done; r.v[GM_HN] = hn;
  unsigned long long c = gm_pub_key(seq), w;
  for (int i = 0; i < GM_PUB; ++i) {
    memcpy(&w, &r.v[i], 8);
    c ^= gm_pub_mix(w, i);
  }
  memcpy(&r.v[GM_PUB], &c, 8);
  return r;
}

int main() {
  std::vector<Rec> old, now;
  const double vals[] = {0.0, 1.0, 2.0, 0.5, 0.25, 1e-9};
  old.push_back(Rec{});   // zeroed memory
  for (int pass = 0; pass < 2; ++pass)
    for (double k : {0.0, 1.0, 2.0, 3.0, 16.0, 17.0, 200.0})
      for (double done : {0.0, 1.0})
        for (double beta : vals)
          for (double res : vals)
            for (double hn : {0.0, 1.0, 0.5, 1e-9})
              (pass ? now : old).push_back(make(beta, res, k, done, hn, pass ? 12 : 10));
  long mixed = 0, wrong = 0, refused = 0;
  double got[GM_PUB];
  for (const Rec& b : now) {
    refused += !gm_pub_read(b.v, b.seq, got) || memcmp(got, b.v, sizeof(got)) != 0;
    for (size_t q = 0; q < old.size(); q += 1) {
      const Rec& a = old[q];
      for (int m = 1; m < 1 << (GM_PUB + 1); ++m) {   // bit i: word i is the old record's
        Rec r = b;
        for (int i = 0; i <= GM_PUB; ++i)
          if (m >> i & 1) r.v[i] = a.v[i];
        if (memcmp(r.v, b.v, sizeof(double) * (GM_PUB + 1)) == 0) continue;   // the stale words are the same
        ++mixed;
        wrong += gm_pub_read(r.v, b.seq, got);
      }
    }
  }
  printf("%ld %ld %ld %zu\n", mixed, wrong, refused, now.size());
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_mixed_up_records_are_refused(tmp_path):
    src = tmp_path / "rec.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "rec"
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=240).stdout.split()
    mixed, wrong, refused, n = map(int, out)
    assert n == 2016 and mixed > 10 ** 8
    assert wrong == 0 and refused == 0
