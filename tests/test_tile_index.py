"""Quotients by a reciprocal that the wave-level linear layer takes its tile from (wgemm.h), against the division, on the host: divisors
and dividends at both ends of 32 bits and around every multiple (no GPU)."""
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_quotients_are_exact_for_all_32_bits(tmp_path):
    src, exe = tmp_path / "q.hip", tmp_path / "q"
    src.write_text('''#include <cstdio>
#include <random>
#include "wgemm.h"
int main() {
  std::mt19937_64 rng(5);
  auto check = [](unsigned int x, unsigned int d) {
    if (df::quotient_u32(x, d, df::reciprocal_u32(d)) != x / d) { printf("%u / %u\\n", x, d); return false; }
    return true;
  };
  for (long long i = 0; i < 3000000; ++i) {
    const int bits = 1 + (int)(rng() % 32);
    unsigned int d = i < 70000 ? (unsigned int)i + 1 : (unsigned int)(rng() >> (64 - bits));
    if (i < 8) d = 0xffffffffu - (unsigned int)i;
    if (d == 0) continue;
    const unsigned int m = 0xffffffffu / d, k = m ? (unsigned int)(rng() % ((unsigned long long)m + 1)) : 0;
    const unsigned int xs[] = {0u, 1u, d - 1, d, d + 1, k * d, k * d - 1, k * d + d - 1, m * d, m * d - 1, 0xffffffffu, 0xfffffffeu, (unsigned int)rng()};
    for (unsigned int x : xs) if (!check(x, d)) return 1;
  }
  printf("ok\\n");
}
''')
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "ok\n"
