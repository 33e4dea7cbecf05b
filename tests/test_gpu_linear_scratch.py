"""Plain packed layers with scratch regions of every size: layers that need theirs are refused below it and run at it; the others run with
any, in no more parts of K than fit."""
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


@pytest.mark.parametrize("M,N,K,due", [
    (1024, 1280, 5120, 3),
    (1632, 1280, 5120, 4),     # whole all the same: the parts were worth it when the set of refusals was fixed
    (1696, 320, 5120, 1),      # five parts, or as many as fit
    (2001, 320, 5120, 1),
    (320, 1920, 5120, 1),
    (2720, 640, 3840, 1),      # two
    (64, 1280, 5120, 1),       # four, or whole
])
def test_linear_packed_scratch_sizes(M, N, K, due):
    x, w = round_bf16(normal(53, "x", (M, K))), round_bf16(normal(53, "w", (N, K), std=1.0 / math.sqrt(K)))
    b, r = normal(53, "b", (N,), std=0.1), normal(53, "r", (M, N))
    xp, wp, bd, rd = df.pack_rows(dev(x, True)), df.pack_linear_weight(dev(w, True)), dev(b), dev(r)
    ref = ops.linear(x, w, b) + r
    part = (M + 31) // 32 * (N // 32) * 4096
    whole = torch.empty(16384 + 8 * part, dtype=torch.uint8, device=xp.device)
    suffices = df.linear_packed_scratch(M, N, xp.device).numel()
    sizes = [16384 + n * part - cut for n in (1, 2, 3, due) for cut in (0, 1)] + [256, 16384, min(suffices, whole.numel())]
    for size in sorted(set(sizes)):
        whole.fill_(255)                                       # NaN where a sum would be missing
        call = lambda: df.linear_packed(xp, wp, M, N, K, bias=bd, residual=rd, want=("f32", "packed", "rows"), scratch=whole[:size])
        if due > 1 and size < 16384 + due * part:
            with pytest.raises(df.DfError):                    # before any launch
                call()
            continue
        outs = call()
        # float sums of K products of size 1 / sqrt(K), in parts: a few ulps of the largest partial sum
        check(host(outs["f32"]), ref, True, "%d x %d x %d in %d bytes" % (M, N, K, size), tol=2e-3, row_tol=8e-3, elt_tol=8e-3, say=say)
        got, _ = unpack_rows(host(outs["packed"]), M, N)
        np.testing.assert_array_equal(got, host(outs["rows"]))
        assert torch.equal(outs["f32"], call()["f32"])
        assert bool((whole[size:] == 255).all()), "written beyond the region"
