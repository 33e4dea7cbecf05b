"""Packed linear layers on tiles, and the fused cross-attention, with K of fewer stages than the operand ring holds, of as many, and of one
more: the stages behind the last request."""
import pytest

from test_gpu_ops import test_cross_attn_packed as run_cross
from test_gpu_ops import test_linear_packed as run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,variant", [
    (4100, 2560, 64, "geglu"),
    (4100, 2560, 128, "ln_geglu"),
    (4100, 2560, 192, "plain"),
    (9000, 1280, 256, "ln"),
    (2100, 1280, 320, "plain"),
    (1100, 640, 128, "plain"),
    (1100, 640, 512, "plain"),
])
def test_linear_of_few_stages(M, N, K, variant):
    run(M, N, K, variant)


@pytest.mark.parametrize("rows,C", [(6000, 128), (6000, 192), (3300, 256)])
def test_cross_attention_of_few_stages(rows, C):
    run_cross(1, rows, C, 77, 2, 1)
