"""Where the row-major tile kernel takes its weights from (tile.h), evaluated on the host for every tile width, both weight layouts and
ragged last tiles (no GPU)."""
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "tile.h"
using namespace df;

int main() {
  const int K = 192, slabs = K / 64;
  long long wrong = 0, n_checked = 0;
  for (int N : {64, 192, 320, 640, 704})
    for (int pad : {0, 8}) {
      const long long ldw = K + pad;
      // every element holds its own number n * K + k, in both layouts
      std::vector<int> rows((size_t)N * ldw, -1), tiles((size_t)N * K, -1);
      for (int n = 0; n < N; ++n)
        for (int k = 0; k < K; ++k) {
          rows[n * ldw + k] = n * K + k;
          const int r = n % 64, slot = (k % 64 / 8) ^ ((r >> 1) & 7);
          tiles[(((size_t)(n / 64) * slabs + k / 64) * 64 + r) * 64 + slot * 8 + k % 8] = n * K + k;
        }
      for (int tiled = 0; tiled < 2; ++tiled)
        for (int bn : {32, 64, 96, 128, 160, 192, 256, 320})
          for (int n0 = 0; n0 < N; n0 += bn)
            for (int row = 0; row < bn; ++row)
              for (int slot = 0; slot < 8; ++slot)
                for (int s = 0; s < slabs; ++s) {
                  const std::vector<int>& w = tiled ? tiles : rows;
                  const size_t at = w_tile_base(tiled, n0, slabs, ldw) + (w_lane_bytes(tiled, n0, row, slot, N, slabs, ldw) + (size_t)s * w_slab_bytes(tiled)) / 2;
                  ++n_checked;
                  if (at + 8 > w.size()) { ++wrong; continue; }                      // out of the weights
                  if (n0 + row >= N) continue;                                       // re-read, never stored
                  const int want = (n0 + row) * K + s * 64 + (slot ^ ((row >> 1) & 7)) * 8;   // the chunk that LDS slot holds
                  for (int e = 0; e < 8; ++e) wrong += w[at + e] != want + e;
                }
    }
  printf("%lld of %lld\n", wrong, n_checked);
  return wrong != 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_tiles_read_their_own_weight_rows(tmp_path):
    src = tmp_path / "addresses.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "addresses"
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
