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


NUMBERS = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "gnmeet.h"

// A slab's words while one call is replayed and others run beside it on another stream, in random order: a workgroup takes its number, publishes,
// and looks; a word with its number has to be of its own launch.  clear: a recorded launch's words are cleared before its workgroups start.
// beside: the other calls, eager ones with numbers of their own.
constexpr int P = 4, LGP = 2;
struct Word { unsigned int tag; int launch; };
struct Group { int pc; unsigned int tag; };
template <typename Number>
long long wrong(std::mt19937& rng, bool clear, bool beside, unsigned int recorded_id, Number number) {
  Word words[P] = {};
  unsigned int tickets = 0;
  unsigned long long calls = 0;
  int launches = 0;
  long long bad = 0;
  struct Launch { int serial; unsigned int id; std::vector<Group> g; bool clear; } run[2] = {};
  for (int step = 0; step < 400; ++step) {
    const int k = beside ? (int)(rng() % 2) : 0;
    Launch& l = run[k];
    std::vector<int> open;
    for (int i = 0; i < (int)l.g.size(); ++i) if (l.g[i].pc < 3) open.push_back(i);
    if (open.empty()) {                                     // the stream's next launch
      l.serial = ++launches;
      l.id = k == 0 ? recorded_id : df::gn_call_id(calls++, false);
      l.g.assign(P, Group{0, 0});
      if (k == 0 && clear) for (Word& w : words) w = Word{0, 0};
      continue;
    }
    const int i = open[rng() % open.size()];
    Group& g = l.g[i];
    if (g.pc == 0) g.tag = number(l.id, tickets++);
    if (g.pc == 1) words[i] = Word{g.tag, l.serial};
    if (g.pc == 2) {
      for (const Word& w : words) bad += w.tag == g.tag && w.launch != l.serial;
      if (rng() % 2) continue;                              // looks again
    }
    ++g.pc;
  }
  return bad;
}

int main() {
  std::mt19937 rng(3);
  auto number = [](unsigned int id, unsigned int ticket) { return df::gn_meet_number(id, ticket, LGP); };
  auto by_ticket = [](unsigned int id, unsigned int ticket) { return id << 16 | (ticket >> LGP & 0xffff); };
  long long plan = 0, lib = 0, tickets = 0, unclear = 0;
  const unsigned int rec = df::gn_call_id(0, true);
  for (int i = 0; i < 20000; ++i) {
    plan += wrong(rng, false, false, 0, number);            // words of a plan's own
    lib += wrong(rng, true, true, rec, number);
    tickets += wrong(rng, false, true, 7000, by_ticket);    // tickets of launches that overlap: not sound
    unclear += wrong(rng, false, true, rec, number);        // nor a recorded call's number alone
  }
  printf("%lld %lld %lld %lld\n", plan, lib, tickets, unclear);
  if (plan || lib || !tickets || !unclear) return 1;
  const unsigned long long M = 0x7fffffffull;
  for (unsigned long long n : {0ull, 1ull, M - 1, M, M + 1, 5 * M - 1, ~0ull}) {
    const unsigned int e = df::gn_call_id(n, false), r = df::gn_call_id(n, true);
    if (!e || e >> 31 || r >> 31 != 1 || df::gn_call_id(n + 1, false) == e || df::gn_call_id(n + 1, true) == r) return 2;
  }
  if (!df::gn_meet_number(0, 0, 1) || !df::gn_meet_number(0, ~0u, 1) || df::gn_meet_number(9, ~0u, 1) != 9) return 3;
  return 0;
}
"""


def test_a_word_counts_in_its_own_launch_only(tmp_path):
    run(tmp_path, NUMBERS)
