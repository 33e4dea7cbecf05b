"""GroupNorms of a plan whose workgroups hand each other their sums, against the same step with workgroups that wait for nobody, or look once or
three times and add up what is missing: the same bits with several segments (the synchronous step), with a concatenation read from its two tensors,
with packed output and boundary rows or columns, and with the cached sums refreshed in place, in every statistic mode, eagerly and replayed."""
import numpy as np
import pytest
import torch

import paper_2402_19481_amd as df
from df_inputs import configs, unet_table as ut
from gpu_util import DEV, dev
from test_gpu_unet import _upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,N,B,cols", [
    (192, 64, 2, 1, False),      # 6144 pixels per patch: both steps meet, the synchronous one in two segments
    (192, 64, 2, 2, False),      # sixteen workgroups a slab
    (256, 64, 4, 1, False),      # four segments
    (256, 96, 8, 2, False),      # eight, of two workgroups each
    (64, 192, 2, 1, True),       # vertical strips: one segment, boundary columns
])
def test_the_bits_do_not_depend_on_who_waits(monkeypatch, H, W, N, B, cols):
    print("plan %d x %d, %d patches, %d items, cols %d" % (H, W, N, B, cols), flush=True)
    monkeypatch.setattr(ut, "SMALL", dict(ut.SMALL, levels=(64, 128, 192), groups=16, depths=(0, 1, 1)))
    cfg = ut.UNetCfg(H=H, W=W, N=N, **ut.SMALL)
    t = configs.unet_inputs(cfg, seed=43, stale_std=0.5)
    many = lambda a: np.concatenate([a] * B)
    x_prev, emb, text = dev(many(t["x_prev"])), dev(many(t["emb"])), dev(many(t["text"]), True)
    patch = N - 1
    x = dev(many(t["x"])).chunk(N, 2 if cols else 1)[patch].contiguous()
    net = df.PatchUNet(cfg, _upload(configs.unet_weights(cfg, seed=43, threads=8)), B=B, device=DEV,
                       split_axis=df.SPLIT_COLS if cols else df.SPLIT_ROWS)

    def results(looks):
        net.set_gn_looks(looks)
        out = []
        net.stale.zero_()
        out += [net.step(x_prev, emb, text, mode=df.MODE_FULL), net.stale.clone()]
        for mode in (df.GN_SUMS, df.GN_EQ2, df.GN_SEPARATE, df.GN_STALE):
            net.set_gn_mode(mode)
            net.stale.copy_(out[1])
            apart = net.step(x, emb, text, patch, df.MODE_DISPLACED, refresh=False)
            out += [net.step(x, emb, text, patch, df.MODE_DISPLACED), net.stale.clone()]
            assert torch.equal(apart, out[-2]), mode               # refreshing the sums in place changes nothing that is read
        return out

    want = results(0)
    assert torch.isfinite(want[0]).all()
    for looks in (-1, 1, 3, 0):
        for k, (a, b) in enumerate(zip(results(looks), want)):
            assert torch.equal(a, b), (looks, k)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):                                     # eager, recorded, replayed
        eps = torch.empty_like(x)
        for rep in range(4):
            for mode, k in ((df.GN_EQ2, 4), (df.GN_SUMS, 2)):
                net.set_gn_looks(1 if rep == 3 else -1)
                net.set_gn_mode(mode)
                net.stale.copy_(want[1])
                net.step(x, emb, text, patch, df.MODE_DISPLACED, out=eps)
                s.synchronize()
                assert torch.equal(eps, want[k]) and torch.equal(net.stale, want[k + 1]), (rep, mode)
    net.close()
