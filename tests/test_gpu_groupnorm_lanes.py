"""GroupNorm with a lane's pixels in registers: the edges between two, four and eight pixels per lane, and more cached entries than a
wave has lanes (the sums of the first 64 come by lane moves, more by a loop)."""
import pytest

import paper_2402_19481_amd as df
from oracle import ops
from gpu_util import TOL_F32, check, dev, host, rel_l2
from test_gpu_ops import _gn_case, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,W,C,G,N,bf16", [
    (4, 51, 1280, 32, 2, False),     # 102 pixels a pass: the most of two, ..
    (5, 41, 1280, 32, 2, True),      # .. one more
    (8, 51, 1280, 32, 2, True),      # the most of four, ..
    (1, 409, 1280, 32, 2, False),    # .. one more
    (4, 102, 320, 32, 2, True),      # 204 pixels a pass, two channels per lane
    (1, 817, 320, 32, 2, False),
    (1, 5, 64, 8, 64, False),        # one cached entry for each lane, ..
    (1, 5, 64, 8, 70, True),         # .. and more than that
])
def test_groupnorm_lane_shares(R, W, C, G, N, bf16):
    for mode, patch in ((0, N - 1), (1, 0), (2, 1), (3, 1)):
        full, st, gamma, beta = _gn_case(11, 2, N * R, W, C, G, N, bf16)
        xf = full[:, patch * R:(patch + 1) * R]
        ref, ref_fs = ops.groupnorm_stale(xf, st, gamma, beta, G, patch, N, 1e-5, mode, True)
        y, fs = df.groupnorm_stale(dev(xf, bf16), dev(st), dev(gamma), dev(beta), G, patch, N, 1e-5, mode, True)
        check(host(y), ref, bf16, "gn %d x %d x %d, %d patches, mode %d" % (R, W, C, N, mode), say=say)
        assert rel_l2(host(fs), ref_fs) < TOL_F32
