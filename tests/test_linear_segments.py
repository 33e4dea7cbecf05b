"""Packed layers whose output is split into segments (queries, keys, values): what the kernels would leave out is refused (wgemm.h, on the
host; no GPU)."""
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_segments_come_alone(tmp_path):
    src, exe = tmp_path / "seg.hip", tmp_path / "seg"
    src.write_text('''#include <cstdio>
#include "wgemm.h"
int main() {
  float x;
  df::WGemmArgs a = {};
  a.ln_s = &x; a.nseg = 3;
  printf("%d", df::segments_alone(a));
  auto with = [&](auto set) { df::WGemmArgs b = a; set(b); printf("%d", df::segments_alone(b)); };
  with([&](df::WGemmArgs& b) { b.residual = &x; });
  with([&](df::WGemmArgs& b) { b.out_f32 = &x; });
  with([&](df::WGemmArgs& b) { b.out_packed = &x; });
  with([&](df::WGemmArgs& b) { b.out_rows = &x; });
  with([&](df::WGemmArgs& b) { b.xa_kv = &x; });
  with([&](df::WGemmArgs& b) { b.geglu = 32; });
  with([&](df::WGemmArgs& b) { b.ln_s = nullptr; });
  with([&](df::WGemmArgs& b) { b.nseg = 0; b.residual = b.out_f32 = &x; b.ln_s = nullptr; });
}
''')
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "100000001"
