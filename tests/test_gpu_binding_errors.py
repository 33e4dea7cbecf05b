"""Errors of torch inside the native binding of the single operations arrive as torch's own."""
import pytest
import torch

import paper_2402_19481_amd as df

pytestmark = pytest.mark.gpu


def test_result_that_does_not_fit():
    x = torch.zeros(1, 64, 256, 2048, dtype=torch.bfloat16, device="cuda:0")       # 64 MB
    g = torch.ones(2048, device="cuda:0")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (1 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            df.groupnorm_stale(x, None, g, g, 32, 0, 1)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    y, fs = df.groupnorm_stale(x, None, g, g, 32, 0, 1)
    assert (y == 1).all() and not fs.any()                     # the shift of a tensor of zeros
