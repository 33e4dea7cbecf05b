"""GroupNorm over a concatenation that is read from its two tensors: groups that cross the border, of 2 to 14 channels, in the
kernel that keeps its pixels in registers, in the two launches, and where the concatenation is written out first (groups of a few small
segments; vertical strips of the whole image).  The bounds are those of the tests that are run, against the oracle."""
import pytest

from df_inputs import unet_table as ut
from test_gpu_unet import test_small_unet_full_and_displaced as run_rows
from test_gpu_unet import test_small_unet_vertical_strips as run_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("run,H,W,N,B", [(run_rows, 16, 8, 2, 2), (run_rows, 64, 40, 2, 1), (run_cols, 8, 16, 2, 2)])
@pytest.mark.parametrize("levels,groups", [((64, 128, 192), 64), ((64, 192, 256), 32)])
def test_concatenation_read_from_two_tensors(monkeypatch, run, H, W, N, B, levels, groups):
    monkeypatch.setattr(ut, "SMALL", dict(ut.SMALL, levels=levels, groups=groups, depths=(0, 1, 1)))
    run(H, W, N, B)
