"""The rules that the workgroups of a GroupNorm go by when they hand each other their sums (gnmeet.h), on the host: every order of their steps, for
launches of two and four workgroups.  A rule that is known to be wrong is tried beside each, which the search has to find out (no GPU)."""
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")


def run(tmp_path, source):
    src, exe = tmp_path / "rules.hip", tmp_path / "rules"
    src.write_text(source)
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


REFRESH = r"""
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>
#include "gnmeet.h"

// A slab's P workgroups: read the cached sums, count themselves, publish, look for the others until all are there or patience ends (at any
// moment), write the patch's own sums.  `base`: the counter of earlier launches.
struct State {
  unsigned char pc[4], arrived[4];
  unsigned char count, published, written;
  bool operator<(const State& o) const { return memcmp(this, &o, sizeof(State)) < 0; }
};
template <typename Rule>
long long wrong(int P, unsigned int base, Rule writes) {
  std::set<State> seen;
  std::vector<State> todo(1);
  memset(&todo[0], 0, sizeof(State));
  long long bad = 0;
  while (!todo.empty()) {
    const State s = todo.back();
    todo.pop_back();
    if (!seen.insert(s).second) continue;
    bool done = true;
    for (int i = 0; i < P; ++i) {
      State n = s;
      if (s.pc[i] < 5) done = false;
      switch (s.pc[i]) {
        case 0: if (s.written) { ++bad; } n.pc[i] = 1; break;                     // reads: the old sums have to be there
        case 1: n.arrived[i] = n.count++; n.pc[i] = 2; break;
        case 2: n.published |= 1 << i; n.pc[i] = 3; break;
        case 3: n.pc[i] = 4; break;                                               // all found, or patience ended
        case 4: if (writes(base + s.arrived[i], P, i)) n.written = 1; n.pc[i] = 5; break;
        default: continue;
      }
      todo.push_back(n);
    }
    if (done && !s.written) ++bad;                                                // somebody has to write them
  }
  return bad;
}

int main() {
  for (int P : {2, 4})
    for (unsigned int base : {0u, 4u, 0xfffffffcu}) {
      if (wrong(P, base, [](unsigned int a, int P, int part) { return df::gn_meet_writes(true, a, P, part); })) return 1;
      if (!wrong(P, base, [](unsigned int, int, int part) { return part == 0; })) return 2;       // the first one, at once: not sound
    }
  if (!df::gn_meet_writes(false, 7, 4, 0) || df::gn_meet_writes(false, 3, 4, 1)) return 3;

  // where a launch without a counter of its own takes the cached sums from a copy: N = 4 patches of n floats, the third is the launch's
  const long long n = 2 * 32 * 2;
  float* s = (float*)4096;
  auto copies = [&](long long at, int mode) { return df::gn_meet_copies(s, s + at, n, 2, 4, mode); };
  for (int mode : {DF_GN_SUMS, DF_GN_EQ2, DF_GN_SEPARATE, DF_GN_STALE}) {
    const bool own = mode == DF_GN_EQ2 || mode == DF_GN_STALE;
    if (copies(2 * n, mode) != own) return 4;
    for (long long at : {0 * n, 1 * n, 3 * n, 2 * n + 1, 2 * n - 1, 4 * n - 1, 1 - n})
      if (!copies(at, mode)) return 5;
    for (long long at : {-n, 4 * n, 9 * n})
      if (copies(at, mode)) return 6;
    if (df::gn_meet_copies(nullptr, s, n, 2, 4, mode) || df::gn_meet_copies(s, nullptr, n, 2, 4, mode)) return 7;
  }
  return 0;
}
"""


def test_own_sums_are_written_when_all_have_read_the_old_ones(tmp_path):
    run(tmp_path, REFRESH)
