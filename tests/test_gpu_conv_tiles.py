"""3x3 convolutions of stride 1 whose input pixels stay in LDS over the taps, against the float64 oracle: every tile shape of the
dispatch, at sizes that leave ragged tiles in both directions of the image and in the output channels."""
import numpy as np
import pytest
import torch

import paper_2402_19481_amd as df
from df_inputs import from_bf16_bits, to_bf16_bits
from gpu_util import check, dev, dev_bits, host
from oracle import ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W,Cin,Cout,N,axis", [
    (1, 8, 7, 64, 32, 2, "rows"),            # 64 pixels x 64 channels, one tile
    (1, 300, 3, 64, 64, 1, "rows"),          # tiles of the whole width
    (2, 12, 12, 640, 320, 4, "cols"),        # ten parts of the channels
    (1, 66, 65, 64, 640, 2, "rows"),         # 128 x 64
    (1, 27, 122, 128, 640, 2, "cols"),
    (1, 18, 37, 1280, 640, 1, "rows"),       # four parts
    (1, 40, 101, 128, 1280, 2, "rows"),      # 256 x 64
    (1, 50, 130, 64, 640, 1, "rows"),        # 128 x 160
    (1, 10, 60, 1280, 1280, 1, "rows"),      # 128 x 128
    (1, 16, 250, 640, 640, 1, "rows"),       # 64 x 160
    (1, 15, 120, 1280, 1280, 1, "rows"),     # 256 x 128
    (1, 250, 260, 64, 160, 1, "rows"),       # 256 x 160
])
def test_conv_resident_pixels(B, H, W, Cin, Cout, N, axis):
    rng = np.random.default_rng(H * W + Cin)
    ax, p = (1, N - 1) if axis == "rows" else (2, N // 2)
    draw = lambda *s: to_bf16_bits(rng.standard_normal(s, dtype=np.float32))
    stale = draw(B, H, W, Cin)
    x = draw(*np.split(stale, N, axis=ax)[p].shape)
    w = to_bf16_bits(rng.standard_normal((Cout, 3, 3, Cin), dtype=np.float32) * np.float32((9 * Cin) ** -0.5))
    b = rng.standard_normal(Cout).astype(np.float32)
    ref = ops.conv3x3_halo(from_bf16_bits(x), from_bf16_bits(stale), from_bf16_bits(w), b, p, N, split_axis=ax)
    conv = df.conv3x3_halo if ax == 1 else df.conv3x3_halo_cols
    got = conv(dev_bits(x), dev_bits(stale), dev_bits(w), dev(b), p, N)
    # rounding to bf16 is off by at most 2^-9 of a value (2^-9 / sqrt(3) in the mean); the float sums of up to 11520 products add
    # less than 1e-5
    check(host(got), ref, True, tol=2e-3, row_tol=4e-3, elt_tol=2.0 ** -8)
