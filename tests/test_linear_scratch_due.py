"""Which plain packed layers refuse a scratch region that is too small (wgemm.h), on the host: the set is part of the entry point's
contract, so both sides of its borders are written down here (no GPU)."""
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build

# N, K: token rows of 32 (first, last, parts the scratch has to hold); everything else runs with any scratch
DUE = {
    (320, 5120): [(103, 112, 3), (123, 168, 2), (205, 210, 4)],
    (640, 3840): [(59, 68, 3), (69, 84, 2), (205, 256, 2)],
    (640, 2560): [(205, 243, 2)],
    (960, 7680): [(16, 16, 8), (17, 20, 6), (21, 21, 5), (51, 64, 2), (65, 68, 5), (69, 84, 4), (85, 90, 3), (129, 168, 2)],
    (1280, 5120): [(25, 32, 3), (33, 48, 2), (51, 52, 4), (103, 128, 2)],
    (1280, 2560): [(103, 121, 2)],
    (1280, 1280): [],
    (1920, 5120): [(25, 32, 2), (35, 35, 4), (69, 84, 2)],
    (2560, 10240): [(5, 8, 6), (9, 12, 4), (13, 16, 3), (17, 24, 2), (25, 32, 4), (33, 40, 3), (49, 64, 2)],
}


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_layers_that_need_their_scratch(tmp_path):
    src, exe = tmp_path / "due.hip", tmp_path / "due"
    src.write_text('#include <cstdio>\n#include "wgemm.h"\nint main() {\n  int n, k;\n  while (scanf("%d %d", &n, &k) == 2)\n'
                   '    for (int mt = 1; mt <= 300; ++mt) printf("%d\\n", df::parts_due(mt, n / 32, k));\n}\n')
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], input="".join("%d %d\n" % s for s in DUE), capture_output=True, text=True, check=True)
    got = list(map(int, out.stdout.split()))
    for i, (shape, spans) in enumerate(DUE.items()):
        want = [next((p for a, b, p in spans if a <= mt <= b), 1) for mt in range(1, 301)]
        assert got[300 * i:300 * i + 300] == want, shape
