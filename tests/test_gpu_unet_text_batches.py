"""UNet steps whose text keys and values are projected from 154 to 308 rows of text with tiled weights: each batch size takes another
output tile, the largest one that is 160 columns wide and so begins in the middle of a 64-row weight tile.  Every batch item has
a text of its own."""
import numpy as np
import pytest

import paper_2402_19481_amd as df
from df_inputs import configs, normal, round_bf16, unet_table as ut
from gpu_util import DEV, TOL_BF16, check, dev, host, rel_l2
from oracle import unet as ounet
from test_gpu_unet import _stale_as_oracle, _upload, check_eps, say

import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [4, 3, 2])
def test_unet_step_of_several_texts(B):
    cfg = ut.UNetCfg(H=16, W=8, N=2, levels=(64, 640), depths=(0, 5), groups=32, emb_dim=128, text_len=77, text_dim=1024,
                     res_per_level=1)
    weights = configs.unet_weights(cfg, seed=21, threads=8)
    t = configs.unet_inputs(cfg, seed=21, stale_std=0.5)
    scale = np.arange(1, B + 1).reshape(B, 1, 1, 1)
    x_prev, x, emb = np.concatenate([t["x_prev"]] * B) * scale, np.concatenate([t["x"]] * B) * scale, np.concatenate([t["emb"]] * B)
    text = round_bf16(normal(21, "texts", (B, cfg.text_len, cfg.text_dim)))
    bl, P, ostale = ut.blocks(cfg), ounet.Params(weights), {}
    net = df.PatchUNet(cfg, _upload(weights), B=B, device=DEV)
    emb_d, text_d = dev(emb), dev(text, True)
    o_full = ounet.unet_step(cfg, bl, P, x_prev, emb, text, ostale, mode=ounet.FULL)
    g_full = host(net.step(dev(x_prev), emb_d, text_d, mode=df.MODE_FULL))
    check_eps(g_full, o_full, "B %d FULL eps" % B)
    for nm in net.stale_names():
        g, o = _stale_as_oracle(net, nm, cfg, B, ostale)
        assert rel_l2(g, o) < TOL_BF16, nm
    # the texts matter by much more than the tolerance
    other = ounet.unet_step(cfg, bl, P, x_prev, emb, text[::-1], {}, mode=ounet.FULL)
    say("  oracle with the texts in another order is", rel_l2(other, o_full), "away")
    assert rel_l2(other, o_full) > 5 * TOL_BF16
    R, stale0 = cfg.H // 2, net.stale.clone()
    for i in range(2):
        net.stale.copy_(stale0)
        xs = x[:, i * R:(i + 1) * R]
        o_disp = ounet.unet_step(cfg, bl, P, xs, emb, text, {k: v.copy() for k, v in ostale.items()}, i, ounet.DISPLACED)
        check_eps(host(net.step(dev(xs), emb_d, text_d, patch_idx=i, mode=df.MODE_DISPLACED)), o_disp, "B %d patch %d eps" % (B, i))
    net.close()
