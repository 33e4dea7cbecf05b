"""Self-attention on either side of the choice between one workgroup per 32 queries (its waves split the keys) and 128 queries per
workgroup: the fewest keys and the most rounds of the first, short and long calls that stay with the second."""
import pytest

from test_gpu_ops import test_attn_stale_vt as run
from test_gpu_ops import test_attn_stale_vt_running_maximum as run_maximum

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Lq,L,heads,packed", [
    (1, 1, 64, 1, False),            # one tile: seven waves without keys
    (2, 33, 65, 3, True),            # a second tile of one key
    (1, 64, 449, 20, True),          # eight tiles, the last of one key
    (1, 128, 1000, 5, False),        # two rounds, a tile of 40 keys last
    (1, 64, 2048, 10, True),         # two blocks: four rounds, the most for them
    (1, 320, 5083, 4, False),        # ten rounds, the most of all
    (1, 33, 64, 129, False),         # 258 blocks of 32 queries: more than one per compute unit
    (2, 96, 200, 43, True),
    (1, 40, 63, 2, False),           # fewer keys than a tile
    (1, 40, 2750, 2, False),         # ranges of keys, the last ragged
    (1, 130, 5700, 3, True),
    (2, 300, 6001, 4, True),
    (1, 512, 8192, 2, False),
])
def test_attn_few_queries(B, Lq, L, heads, packed):
    run(B, Lq, L, heads, packed)


@pytest.mark.parametrize("Lq,L,heads", [(129, 65, 52), (31, 127, 257), (257, 129, 29), (300, 449, 26), (40, 2750, 2)])
@pytest.mark.parametrize("shape", ["rising", "falling", "spike"])
def test_attn_running_maximum_more_heads(Lq, L, heads, shape):
    run_maximum(Lq, L, heads, shape)
