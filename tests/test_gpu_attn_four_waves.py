"""Self-attention of few queries whose blocks are counted head by head: 257 to 512 blocks of 32 queries (four waves each), and fewer of
them where the heads do not divide among the XCDs (eight waves)."""
import pytest

from test_gpu_ops import test_attn_stale_vt as run
from test_gpu_ops import test_attn_stale_vt_running_maximum as run_maximum

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Lq,L,heads,packed", [
    (1, 31, 64, 257, False),         # one tile: 128 queries per workgroup
    (1, 31, 250, 259, False),        # one block a head, a tile a wave; the XCDs share them unevenly
    (1, 500, 190, 31, True),         # fewer tiles than waves
    (1, 416, 416, 20, True),         # 260 blocks of 13 a head, seven tiles: a wave with one, the last ragged
    (3, 97, 449, 23, True),          # batch items in the count, a last tile of one key, a last block of one query
    (2, 250, 500, 20, False),
    (1, 512, 577, 32, True),         # 512 blocks: the most
    (1, 513, 577, 32, False),        # and 544: 128 queries per workgroup
    (1, 1024, 64, 16, False),
    (1, 352, 704, 20, True),         # eight waves, 33 blocks on an XCD head by head
    (2, 185, 513, 20, False),
    (1, 896, 449, 9, True),
])
def test_attn_blocks_head_by_head(B, Lq, L, heads, packed):
    run(B, Lq, L, heads, packed)


@pytest.mark.parametrize("Lq,L,heads", [(129, 449, 53), (31, 449, 300), (352, 577, 20)])
@pytest.mark.parametrize("shape", ["rising", "falling", "spike"])
def test_attn_running_maximum_head_by_head(Lq, L, heads, shape):
    run_maximum(Lq, L, heads, shape)
