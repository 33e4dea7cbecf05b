"""Plain linear layers of few tokens and a long K on the wave-level kernel in four parts of K: one row to three fragment rows, k-steps
in fives and in fours; and the same layer whole, where the scratch does not hold the sums."""
import math

import numpy as np
import pytest
import torch

import paper_2402_19481_amd as df
from df_inputs import normal, round_bf16
from gpu_util import check, dev, host
from oracle import ops
from test_gpu_ops import say, unpack_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 1280, 5120), (64, 1280, 5120), (96, 1280, 5120), (33, 640, 4096), (40, 64, 6144)])
def test_linear_packed_parts_few_tokens(M, N, K):
    x, w = round_bf16(normal(47, "x", (M, K)) + 0.3), round_bf16(normal(47, "w", (N, K), std=1.0 / math.sqrt(K)))
    b, r = normal(47, "b", (N,), std=0.1), normal(47, "r", (M, N))
    xp, wp, bd, rd = df.pack_rows(dev(x, True)), df.pack_linear_weight(dev(w, True)), dev(b), dev(r)
    scratch = df.linear_packed_scratch(M, N, xp.device)
    ref = ops.linear(x, w, b) + r
    # float sums of K products of size 1 / sqrt(K), in parts: a few ulps of the largest partial sum
    for scr in (scratch, scratch[:16384], None):       # parts; whole: too little scratch, none
        if scr is not None:
            scr.fill_(255)                             # NaN where a sum would be missing
        outs = df.linear_packed(xp, wp, M, N, K, bias=bd, residual=rd, want=("f32", "packed", "rows"), scratch=scr)
        check(host(outs["f32"]), ref, True, "parts of few tokens %d x %d x %d" % (M, N, K), tol=2e-3, row_tol=8e-3, elt_tol=8e-3, say=say)
        got, _ = unpack_rows(host(outs["packed"]), M, N)
        np.testing.assert_array_equal(got, host(outs["rows"]))
        again = df.linear_packed(xp, wp, M, N, K, bias=bd, residual=rd, want=("f32",), scratch=scr)
        assert torch.equal(outs["f32"], again["f32"])
