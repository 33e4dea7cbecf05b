"""Packed linear layers on tiles, and the fused cross-attention, with K of fewer stages than the operand ring holds, of as many, and of one
more: the stages behind the last request.  The tile of each row is asserted by test_linear_choice.py."""
import pytest

from test_gpu_ops import test_cross_attn_packed as run_cross
from test_gpu_ops import test_linear_packed as run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,variant", [
    (4100, 2560, 64, "geglu"),         # 128 x 128, a ring of two stages: one, two
    (4100, 2560, 128, "ln_geglu"),
    (4100, 2560, 192, "plain"),        # 128 x 192, six stages in a ring of six; two and four
    (2708, 1920, 64, "plain"),
    (915, 5120, 128, "plain"),
    (2100, 1280, 320, "plain"),        # 128 x 96, five in five
    (1100, 640, 128, "plain"),         # 64 x 64, one to four in four
    (1100, 640, 512, "plain"),
    (1100, 640, 128, "ln"),
    (1100, 640, 256, "ln"),
    (1100, 640, 384, "ln"),
    (1100, 640, 512, "ln"),
    (8250, 960, 128, "geglu"),         # 128 x 320, four and six in five; pairs that two waves share
    (8250, 960, 128, "ln_geglu"),
    (8250, 960, 192, "ln_geglu"),
    (1567, 10240, 128, "ln_geglu"),    # 256 x 320, four in four
    (2056, 960, 320, "ln_geglu"),      # 128 x 128, five in four
    (9000, 1280, 256, "ln"),           # the wave-level kernel
])
def test_linear_of_few_stages(M, N, K, variant):
    run(M, N, K, variant)


@pytest.mark.parametrize("rows,C,text", [
    (6000, 128, 77), (6000, 192, 77), (3300, 256, 77),         # the wave-level kernel
    (8250, 256, 77),                   # 128 x 128, two workgroups per unit: four stages in a ring of two
    (4664, 448, 77),                   # 128 x 128 in a ring of four, seven stages; its keys come beside the last one
    (4012, 512, 77),
    (3034, 640, 77),
    (4012, 512, 33),                   # 64 x 128, two k-groups that add their sums in LDS: eight and ten stages in three
    (3034, 640, 128),
    (1224, 1280, 50),
])
def test_cross_attention_of_few_stages(rows, C, text):
    run_cross(1, rows, C, text, 2, 1)
