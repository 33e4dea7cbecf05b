"""Packed linear layers on the 64 x 96, 128 x 160, 256 x 256, 128 x 96 and 128 x 192 tiles of bgemm.hip, at sizes the dispatch gives
to them (asserted by test_linear_choice.py), with a ragged last tile along the tokens and, where the width allows, along the features."""
import pytest

from test_gpu_ops import test_linear_packed as run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,variant", [
    (919, 1280, 640, "plain"),         # 64 x 96, 40 feature fragments in tiles of three
    (1590, 960, 640, "ln"),
    (2200, 1920, 384, "plain"),        # 128 x 160
    (1651, 2560, 640, "ln"),
    (5000, 2560, 128, "plain"),        # 256 x 256
    (1241, 10240, 320, "ln_geglu"),
    (1224, 1920, 128, "plain"),        # 128 x 96
    (1102, 2560, 384, "ln"),
    (919, 5120, 128, "plain"),         # 128 x 192
    (1131, 5120, 640, "ln_geglu"),
    (1163, 3840, 384, "ln_geglu"),     # 128 x 128, two workgroups per unit
    (2444, 5120, 256, "ln_geglu"),
])
def test_linear_packed_more_tiles(M, N, K, variant):
    run(M, N, K, variant)
