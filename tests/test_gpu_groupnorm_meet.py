"""GroupNorm in one launch whose workgroups hand each other their sums: the sizes between a workgroup per group and two launches, the edges of
a workgroup's share, every statistic mode, and the same bits where no workgroup waits for another, in a replayed graph and on two streams."""
import numpy as np
import pytest
import torch

import paper_2402_19481_amd as df
from oracle import ops
from gpu_util import TOL_F32, check, dev, host, rel_l2
from test_gpu_ops import _gn_case, say

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("R,W,C,G,N,bf16,B", [
    (1, 817, 320, 32, 2, False, 2),    # the fewest pixels of the form; five lanes a pixel over a group's edge
    (26, 19, 1280, 32, 2, True, 1),    # ragged
    (7, 409, 640, 32, 4, True, 2),     # 2863 pixels over sixteen workgroups, the last with fewer
    (8, 1632, 320, 32, 2, False, 1),   # 32 workgroups of 102 pixels at once: the most of four pixels per lane, ..
    (8, 1637, 320, 32, 2, False, 1),   # .. more,
    (12, 2176, 320, 32, 2, False, 1),  # the most of eight, ..
    (1, 26113, 320, 32, 2, False, 1),  # .. and one more: two launches
    (8, 1632, 320, 32, 2, True, 1),    # two pixels of five lanes
    (40, 30, 2560, 32, 16, False, 1),  # the most cached entries
    (33, 64, 256, 16, 2, True, 1),     # two groups a slab
    (64, 64, 128, 8, 3, False, 3),     # one
    (33, 64, 256, 64, 2, False, 1),    # eight: not this form
])
def test_groupnorm_meeting_workgroups(R, W, C, G, N, bf16, B):
    for mode, patch in ((0, N - 1), (1, 0), (2, 1), (3, 1)):
        full, st, gamma, beta = _gn_case(17, B, N * R, W, C, G, N, bf16)
        xf = full[:, patch * R:(patch + 1) * R]
        ref, ref_fs = ops.groupnorm_stale(xf, st, gamma, beta, G, patch, N, 1e-5, mode, True)
        args = (dev(xf, bf16), dev(st), dev(gamma), dev(beta), G, patch, N, 1e-5, mode, True)
        y, fs = df.groupnorm_stale(*args)
        check(host(y), ref, bf16, "gn %d x %d x %d, %d patches, mode %d" % (R, W, C, N, mode), say=say)
        assert rel_l2(host(fs), ref_fs) < TOL_F32
        alone, fs_alone = df.groupnorm_stale_alone(*args)      # every workgroup adds up all ranges itself
        assert torch.equal(_bits(y), _bits(alone)) and torch.equal(fs, fs_alone)


def test_groupnorm_sums_refreshed_in_place():
    """The patch's own cached sums are written while other workgroups of the launch need the old ones."""
    N, patch = 4, 2
    full, st, gamma, beta = _gn_case(19, 1, N * 32, 64, 640, 32, N, True)
    x = dev(full[:, patch * 32:(patch + 1) * 32], True)
    cache = dev(st)
    for mode in (1, 3):                                        # (modes that read the own entry)
        y0, fs0 = df.groupnorm_stale(x, dev(st), dev(gamma), dev(beta), 32, patch, N, 1e-5, mode, True)
        cache.copy_(dev(st))
        y, fs = df.groupnorm_stale(x, cache, dev(gamma), dev(beta), 32, patch, N, 1e-5, mode, True, fresh_stats_out=cache[patch])
        assert torch.equal(_bits(y), _bits(y0)) and torch.equal(cache[patch], fs0)
        assert torch.equal(cache[[0, 1, 3]], dev(st)[[0, 1, 3]])


@pytest.mark.parametrize("B", [1, 3])
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_groupnorm_sums_refreshed_in_place_by_nobody_who_waits(mode, B):
    """The same, and no workgroup knows of another: the old sums are still those that all of them read."""
    N, patch = 4, 2
    full, st, gamma, beta = _gn_case(31, B, N * 32, 64, 640, 32, N, True)
    x = dev(full[:, patch * 32:(patch + 1) * 32], True)
    args = (dev(gamma), dev(beta), 32, patch, N, 1e-5, mode, True)
    y0, fs0 = df.groupnorm_stale(x, dev(st), *args)
    for call in (df.groupnorm_stale, df.groupnorm_stale_alone):
        cache = dev(st)
        y, fs = call(x, cache, *args, fresh_stats_out=cache[patch])
        assert torch.equal(_bits(y), _bits(y0)) and torch.equal(cache[patch], fs0)
        assert torch.equal(cache[[0, 1, 3]], dev(st)[[0, 1, 3]])
    cache, y = dev(st), torch.empty_like(x)                    # and by the entry point that allocates nothing
    df.groupnorm_stale_noalloc(x, cache, dev(gamma), dev(beta), 32, patch, N, y, cache[patch], 1e-5, mode, True)
    assert torch.equal(_bits(y), _bits(y0)) and torch.equal(cache[patch], fs0)


def test_groupnorm_replays_and_streams():
    N, patch = 2, 1
    cases = []
    for seed, (R, W, C) in enumerate([(32, 32, 1280), (40, 50, 320), (26, 19, 1920)]):
        full, st, gamma, beta = _gn_case(23 + seed, 1, N * R, W, C, 32, N, True)
        cases.append((dev(full[:, R:], True), dev(st), dev(gamma), dev(beta), 32, patch, N, 1e-5, 0, True))
    want = [df.groupnorm_stale(*c) for c in cases]
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        outs = [df.groupnorm_stale(*c) for c in cases]
    for rep in range(4):
        for y, fs in outs:
            y.fill_(float("nan")); fs.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            g.replay()
        torch.cuda.synchronize()
        for (y, fs), (y0, fs0) in zip(outs, want):
            assert torch.equal(_bits(y), _bits(y0)) and torch.equal(fs, fs0), rep
        df.groupnorm_stale(*cases[rep % 3])                    # other calls between the replays
    streams = [torch.cuda.Stream() for _ in range(4)]
    got = []
    for rep in range(8):
        for s in streams:
            with torch.cuda.stream(s):
                got.append((rep % 3, df.groupnorm_stale(*cases[rep % 3])))
    torch.cuda.synchronize()
    for k, (y, fs) in got:
        assert torch.equal(_bits(y), _bits(want[k][0])) and torch.equal(fs, want[k][1])


def test_groupnorm_replays_beside_other_calls():
    """A recorded call on new values each time, while calls of the same size run on another stream (and share its words now and then)."""
    N, patch, R, W, C = 2, 1, 32, 32, 1280
    full, st, gamma, beta = _gn_case(37, 1, N * R, W, C, 32, N, True)
    args = (dev(st), dev(gamma), dev(beta), 32, patch, N, 1e-5, 0, True)
    xs = [dev(full[:, R:] * (1 + k), True) for k in range(3)]
    want = [df.groupnorm_stale(x, *args) for x in xs]
    buf, one, two = xs[0].clone(), torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=one):
        y, fs = df.groupnorm_stale(buf, *args)
    got, other = [], []
    for rep in range(24):
        with torch.cuda.stream(two):
            other += [(k, df.groupnorm_stale(xs[k], *args)) for k in range(3)]
        with torch.cuda.stream(one):
            buf.copy_(xs[rep % 3])
            g.replay()
            got.append((rep % 3, (y.clone(), fs.clone())))
    torch.cuda.synchronize()
    for k, (yy, ff) in got + other:
        assert torch.equal(_bits(yy), _bits(want[k][0])) and torch.equal(ff, want[k][1]), k


def test_groupnorm_beside_a_kernel_that_holds_units():
    """Eight pixels per lane, so a workgroup needs a unit's registers: those of units that another stream's kernel holds start when others have left,
    which add up the missing ranges."""
    N, patch = 2, 1
    full, st, gamma, beta = _gn_case(41, 1, N * 64, 256, 960, 32, N, True)
    args = (dev(full[:, 64:], True), dev(st), dev(gamma), dev(beta), 32, patch, N, 1e-5, 0, True)
    y0, fs0 = df.groupnorm_stale_alone(*args)
    streams = [torch.cuda.Stream() for _ in range(3)]
    for blocks in (8, 100, 250):
        got = []
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[0]):
            df.mfma_probe(blocks, 20000)                       # (0.5 ms)
        for s in streams[1:]:                                  # (one of them may share the hardware queue of the first)
            with torch.cuda.stream(s):
                got += [df.groupnorm_stale(*args) for _ in range(4)]
        torch.cuda.synchronize()
        for y, fs in got:
            assert torch.equal(_bits(y), _bits(y0)) and torch.equal(fs, fs0), blocks


def test_groupnorm_in_place():
    """y over x: the form whose workgroups might read it again is not taken."""
    full, st, gamma, beta = _gn_case(29, 1, 2 * 32, 32, 1280, 32, 2, True)
    x = dev(full[:, 32:], True)
    args = (dev(st), dev(gamma), dev(beta), 32, 1, 2)
    ref, ref_fs = ops.groupnorm_stale(full[:, 32:], st, gamma, beta, 32, 1, 2, 1e-5, 0, False)
    fs = torch.empty(1, 32, 2, device=x.device)
    df.groupnorm_stale_noalloc(x, *args, x, fs)
    check(host(x), ref, True, "gn in place", say=say)
    assert rel_l2(host(fs), ref_fs) < TOL_F32
    np.testing.assert_array_equal(np.isfinite(host(fs)), True)
