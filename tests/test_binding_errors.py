"""What the native binding of the single operations refuses, and how (no GPU: nothing is launched)."""
import pytest
import torch

import paper_2402_19481_amd as df

X = torch.zeros(1, 8, 8, 32)


@pytest.mark.parametrize("call,error", [
    (lambda: df.groupnorm_stale(X, None, X, X, 8, 0, 1), df.DfError),                         # not on the GPU
    (lambda: df.buffer_refresh(X, X, 0, 2), df.DfError),
    (lambda: df.attn_displaced(X[0], X, X, X, X, 2, 0, 1), df.DfError),
    (lambda: df.linear(X.view(64, 32), X, out_dtype=torch.float16), df.DfError),              # type of the result
    (lambda: df.groupnorm_stale(X[0], None, X, X, 8, 0, 1), ValueError),                      # dimensions
    (lambda: df.conv3x3_halo_cols(X[0], None, X, None, 0, 1), ValueError),
    (lambda: df.attn_displaced_cols(X, X, X, X, X, 2, 8, 8, 0, 1), ValueError),
    (lambda: df.linear(X, X), ValueError),
    (lambda: df.conv3x3_halo(X, None, X, None, 0, 1, stride=0), ZeroDivisionError),
    (lambda: df.linear(3, X), TypeError),
    (lambda: df.groupnorm_stale(X, None, X, X, "8", 0, 1), TypeError),
])
def test_refusals(call, error):
    with pytest.raises(error):
        call()
