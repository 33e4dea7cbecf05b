"""Packed linear layers of so many tokens that groups of token rows squared no longer fit 32 bits: the widths and K that always go to the
wave-level kernel."""
import numpy as np
import pytest
import torch

import paper_2402_19481_amd as df
from gpu_util import check, host
from oracle import ops
from test_gpu_ops import DEV, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(2097120, 32, 64), (2097121, 32, 64), (1300011, 96, 64)])
def test_linear_packed_of_millions_of_tokens(M, N, K):
    say("linear of millions of tokens", M, N, K)
    g = torch.Generator(device=DEV).manual_seed(67)
    x = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g, device=DEV) * K ** -0.5).to(torch.bfloat16)
    b = torch.randn(N, generator=g, device=DEV)
    out = df.linear_packed(df.pack_rows(x), df.pack_linear_weight(w), M, N, K, bias=b)["f32"]
    # float sums of 64 products of size 1 / 8: a few ulps of values up to 6
    assert float((out - (x.float() @ w.float().T + b)).abs().max()) < 1e-4
    rows = np.unique(np.concatenate([np.arange(40), np.arange(M - 70, M), np.random.default_rng(1).integers(0, M, 2000)]))
    rows = torch.from_numpy(rows).to(DEV)
    check(host(out[rows]), ops.linear(host(x[rows]).astype(np.float32), host(w).astype(np.float32), host(b)), False, "rows", say=say)
