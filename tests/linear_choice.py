"""The kernel that runs a packed linear layer (wchoice.h), asked on the host: a small program around the header, built once per run."""
import functools
import os
import subprocess
import tempfile

from paper_2402_19481_amd import build

WAVE = "wave"
# tiles of kTiles (tokens x features, k-groups, ring stages), "/2" where two workgroups share a unit
TILES = ["256x320", "128x128/2", "128x128", "64x128/2", "64x64/2", "64x64", "128x320", "64x96", "128x160", "256x256", "128x96", "128x192"]

SOURCE = r'''#include <cstdio>
#include "wchoice.h"
int main() {
  int M, N, K, ln, geglu, nseg, text; long long room;
  while (scanf("%d %d %d %d %d %d %d %lld", &M, &N, &K, &ln, &geglu, &nseg, &text, &room) == 8) {
    df::WParams p = {};
    static float one;
    p.M = M; p.K = K; p.geglu = geglu; p.N = geglu ? N / 2 : N; p.nseg = nseg;
    if (ln) p.ln_s = &one;
    if (text) { p.xkv = reinterpret_cast<const df::bf16x8*>(&one); p.xa_keys = text; }
    int parts = 1;
    const int tile = df::choose_tile(p, df::wave_form(p), room, &parts);
    printf("%d %d\n", tile, parts);
  }
}
'''


@functools.lru_cache(None)
def _program():
    d = tempfile.mkdtemp()
    src, exe = os.path.join(d, "choice.hip"), os.path.join(d, "choice")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["hipcc", *build.FLAGS, "-I", build.CSRC, src, "-o", exe], check=True, capture_output=True)
    return exe


def choices(layers):
    """layers: (M, N, K, variant[, n]); variant: words of ln, geglu, qkv, xa joined by "_", or plain; n: with xa the text tokens (77), else
    the parts of K that fit the scratch (0).  Returns (tile name or WAVE, parts) of each."""
    lines = []
    for M, N, K, variant, *n in layers:
        v = variant.split("_")
        ln, text = bool({"ln", "qkv", "xa"} & set(v)), (n[0] if n else 77) if "xa" in v else 0
        lines.append("%d %d %d %d %d %d %d %d" % (M, N, K, ln, "geglu" in v, 3 * ("qkv" in v), text, n[0] if n and not text else 0))
    out = subprocess.run([_program()], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split()
    return [(WAVE if int(t) < 0 else TILES[int(t)], int(n)) for t, n in zip(out[::2], out[1::2])]
