"""The wave-level packed linear layer at the ends of its index arithmetic: one group of token rows, one k-step per wave, a K loop of one
and of two rounds of the operand ring, and every kind of output with them."""
import numpy as np
import pytest

from test_gpu_ops import test_linear_packed as run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,variant", [
    (1, 64, 64, "plain"),              # one token, one k-fragment per wave
    (32, 32, 64, "ln"),                # one workgroup
    (33, 128, 64, "geglu"),
    (20, 320, 320, "plain"),           # the ring filled once, nothing to refill
    (40, 320, 640, "ln_geglu"),        # filled twice
    (64, 1280, 256, "ln"),             # four k-steps a wave
    (350, 2560, 128, "geglu"),         # 64 x 64 tiles, two k-steps a wave
    (4097, 64, 64, "plain"),           # many groups of token rows
])
def test_wave_level_edges(M, N, K, variant):
    run(M, N, K, variant)
