"""The GroupNorm's division by a reciprocal and reciprocal square root (common.h), on the host: the bits of a division, the rounding of
double (no GPU)."""
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include "common.h"

int main() {
  std::mt19937_64 g(1);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  const double inf = INFINITY;
  long long differ = 0;
  double worst = 0.0;
  for (int i = 0; i < 4000000; ++i) {
    const double n = (double)(1 + g() % (1ull << (1 + i % 40))), s = std::ldexp(u(g), (int)(g() % 200) - 100);
    differ += df::div_by(s, n, 1.0 / n) != s / n;
    const double v = std::ldexp(1.0 + std::fabs(u(g)), (int)(g() % 198) - 99);
    const float e = (float)(1.0 / std::sqrt(v));
    for (float r : {std::nextafterf(e, 0.f), e, std::nextafterf(e, 1e38f)})         // the estimate is off by an ulp
      worst = std::fmax(worst, std::fabs((double)(df::rsqrt_from(v, r) * sqrtl((long double)v) - 1.0L)));
  }
  differ += df::div_by(inf, 3.0, 1.0 / 3.0) != inf || df::div_by(-inf, 3.0, 1.0 / 3.0) != -inf || df::div_by(0.0, 3.0, 1.0 / 3.0) != 0.0;
  differ += !std::isnan(df::div_by(NAN, 3.0, 1.0 / 3.0));
  printf("%lld quotients differ, reciprocal square root off by %g\n", differ, worst);
  return differ != 0 || !(worst < 2.3e-16);          // 2^-53 of v * r, half of it in r, and 2^-53 of the last sum: 1.7e-16
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_quotients_and_reciprocal_square_roots(tmp_path):
    src, exe = tmp_path / "helpers.hip", tmp_path / "helpers"
    src.write_text(PROGRAM)
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
