"""Packed linear layers whose epilogue runs in the accumulators (one k-group): pairs that two waves share, ragged tiles, every output
form, and the form with a single packed output.  The tile of each row is asserted by test_linear_choice.py."""
import numpy as np
import pytest

import paper_2402_19481_amd as df
from df_inputs import normal, round_bf16
from oracle import ops
from gpu_util import check, dev, host
from test_gpu_ops import say, unpack_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,ln", [
    (300, 10240, 1280, True),          # 128 x 128: a value and its gate per wave
    (993, 10240, 640, True),           # 128 x 320: the odd pair is shared
    (1763, 5184, 640, True),           # a last tile of one pair, its neighbours beyond the width
    (4065, 5120, 640, True),           # 256 x 320, two token rows per wave
    (4065, 5120, 640, False),          # bias in place of the norm
    (2590, 5120, 640, True),           # 256 x 256
    (494, 10240, 1280, False),         # 128 x 192: one pair and a share of the next
    (494, 10240, 1280, True),
    (1131, 5120, 640, True),
])
def test_geglu_in_the_accumulators(M, N, K, ln):
    say("geglu epilogue", M, N, K, ln)
    x = round_bf16(normal(61, "x", (M, K)) + 0.3)
    w = round_bf16(normal(61, "w", (N, K), std=K ** -0.5))
    s, t = w.astype(np.float64).sum(1).astype(np.float32), normal(61, "t", (N,), std=0.1)
    pre = x.astype(np.float64) @ w.astype(np.float64).T
    if ln:
        xd = x.astype(np.float64)
        mean, var = xd.mean(1, keepdims=True), xd.var(1, keepdims=True)
        pre = (pre - mean * s) / np.sqrt(var + 1e-5)
    ref = ops.geglu(pre + t)
    kw = dict(ln_s=dev(s), ln_t=dev(t), ln_eps=1e-5) if ln else dict(bias=dev(t))
    xp, wp = df.pack_rows(dev(x, True)), df.pack_linear_weight(dev(w, True))
    outs = df.linear_packed(xp, wp, M, N, K, geglu=True, want=("f32", "packed", "rows"), **kw)
    check(host(outs["f32"]), ref, True, "geglu f32", tol=2e-3, row_tol=8e-3, elt_tol=8e-3, say=say)
    got, _ = unpack_rows(host(outs["packed"]), M, N // 2)
    np.testing.assert_array_equal(got, host(outs["rows"]))
    alone = df.linear_packed(xp, wp, M, N, K, geglu=True, want=("packed",), **kw)["packed"]
    np.testing.assert_array_equal(host(alone), host(outs["packed"]))
