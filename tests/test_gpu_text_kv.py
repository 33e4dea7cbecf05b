"""Text keys / values projected straight into the fragments of the cross-attention, against the projection followed by its packing.  Whole
numbers whose sums stay below 2^24: both sides add exactly and round once, so every bit is the same."""
import pytest
import torch

import paper_2402_19481_amd as df
from test_gpu_ops import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,TL,K,C,count", [
    (1, 1, 64, 64, 1),                # one slab, one tile
    (1, 77, 128, 64, 3),              # the loads of a tile are all out before its first product
    (1, 77, 2048, 640, 10),           # fewer tiles than compute units
    (1, 77, 320, 1280, 21),           # some workgroups with a second tile, five slabs
    (1, 32, 192, 320, 120),           # three tiles each, not all
    (1, 33, 256, 128, 2),
    (1, 96, 256, 192, 3),             # a tile with keys and values
    (1, 128, 448, 128, 4),
    (2, 77, 256, 1280, 30),           # two items of a pass
    (2, 64, 128, 64, 1),
    (2, 128, 320, 320, 2),
    (2, 5, 64, 320, 60),
    (3, 77, 256, 128, 3),             # the last pass has one item
    (4, 100, 192, 640, 40),
])
def test_text_kv(B, TL, K, C, count):
    say("text_kv", B, TL, K, C, count)
    g = torch.Generator(device="cpu").manual_seed(7)
    x = torch.randint(-8, 9, (B * TL, K), generator=g).to(torch.bfloat16).cuda()
    w = torch.randint(-8, 9, (count * 2 * C, K), generator=g).to(torch.bfloat16).cuda()
    shape = (B, count, C // 64, 3, -1)
    want = df.pack_text_kv(df.linear(x, w), B, TL, count, C).view(torch.int16).view(shape)
    got = df.text_kv(x, w, B, TL, count, C).view(torch.int16).view(shape)
    assert torch.equal(got[..., :2, :], want[..., :2, :])       # keys and values; the last third of a head is not used


def test_text_kv_refuses():
    x, w = torch.zeros(129, 64, dtype=torch.bfloat16).cuda(), torch.zeros(128, 64, dtype=torch.bfloat16).cuda()
    with pytest.raises(df.DfError):
        df.text_kv(x, w, 1, 129, 1, 64)
    with pytest.raises(df.DfError):
        df.text_kv(torch.zeros(4, 96, dtype=torch.bfloat16).cuda(), torch.zeros(128, 96, dtype=torch.bfloat16).cuda(), 1, 4, 1, 64)
