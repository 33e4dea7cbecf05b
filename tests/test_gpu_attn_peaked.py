"""Attention whose scores spread over tens of nats, so that tiles of keys hold probabilities far above 1 relative to the maximum of the tiles
before them: against the oracle, and the time it takes beside flat scores."""
import numpy as np
import pytest
import torch

import paper_2402_19481_amd as df
from df_inputs import normal, round_bf16
from gpu_util import DEV, check, dev, host
from oracle import ops
from test_gpu_ops import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["vt", "vt scaled", "rows", "cols"])
@pytest.mark.parametrize("H,N,std", [(257, 3, 4.0), (256, 3, 8.0), (257, 3, 20.0), (43, 3, 8.0)])
def test_attention_peaked_scores(H, N, std, form):
    say("attention_peaked", H, N, std, form)
    heads, L, Lq = 8, H * N, H
    C = heads * 64
    unit = 0.125 * np.log2(np.e) if form == "vt scaled" else 1.0
    q, k = round_bf16((std * unit * normal(71, "q", (1, Lq, C))).astype(np.float32)), round_bf16(normal(71, "k", (1, L, C)))
    v = round_bf16(normal(71, "v", (1, L, C)))
    ref = ops.attention_dense(q.astype(np.float64) / unit, k, v, heads)
    qd, kd, vd = dev(q, True), dev(k, True), dev(v, True)
    if form.startswith("vt"):
        qd = qd.repeat(1, -(-33 * 32 // Lq), 1)            # (more query blocks than the form for few queries takes)
        vt = torch.full((1, C, (L + 63) // 64 * 64), float("nan"), dtype=torch.bfloat16, device=DEV)
        vt[:, :, :L] = vd.transpose(1, 2)
        got = host(df.attn_stale_vt(qd, kd, vt, heads, L, scale=float(np.log(2)) if form == "vt scaled" else None))
        for part in range(0, got.shape[1], Lq):
            check(got[:, part:part + Lq], ref, True, "attention_peaked", say=say)
        return
    if form == "rows":
        own = slice(Lq, 2 * Lq)
        got = host(df.attn_displaced(qd, kd[:, own].contiguous(), vd[:, own].contiguous(), kd, vd, heads, 1, N))
    else:
        got = host(df.attn_displaced_cols(qd, kd[:, 1::3].contiguous(), vd[:, 1::3].contiguous(), kd, vd, heads, H, 3, 1, N))
    check(got, ref, True, "attention_peaked", say=say)


@pytest.mark.parametrize("form", ["vt", "rows"])
@pytest.mark.parametrize("top", [25.0, 27.0])
def test_attention_peaked_scores_beyond_24_bits(form, top):
    """Scores of 1.7e7 nats (2.4e7 in powers of two, where floats are 2 apart) and one key, in the third tile, 34 or 38 nats above all others:
    the tile is scaled by 2^-49 or 2^-55, the maximum can only move by 48 or 56.  The result is that key's values.  The products are
    whole multiples of 16 below 2^27, so their sums are exact."""
    say("attention_peaked beyond 24 bits", form, top)
    heads, Lq, N = 8, 257, 3
    C, L = heads * 64, Lq * N
    q, k = np.full((1, Lq, C), 2048.0, np.float32), np.full((1, L, C), 1024.0, np.float32)
    q[:, :, ::64], k[:, :, ::64], k[:, 150, ::64] = 16.0, 8.0, top
    v = round_bf16(normal(74, "v", (1, L, C)))
    ref = ops.attention_dense(q, k, v, heads)
    qd, kd, vd = dev(q, True), dev(k, True), dev(v, True)
    if form == "vt":
        vt = torch.zeros((1, C, (L + 63) // 64 * 64), dtype=torch.bfloat16, device=DEV)
        vt[:, :, :L] = vd.transpose(1, 2)
        got = host(df.attn_stale_vt(qd.repeat(1, 5, 1), kd, vt, heads, L))[:, :Lq]
    else:
        own = slice(Lq, 2 * Lq)
        got = host(df.attn_displaced(qd, kd[:, own].contiguous(), vd[:, own].contiguous(), kd, vd, heads, 1, N))
    check(got, ref, True, "attention_peaked", say=say)


def test_attention_peaked_scores_take_no_detour():
    """1024 queries x 4096 keys x 10 heads: 25 us with flat scores; 31 where a tile with large probabilities is scaled in registers, 43
    where every such tile is computed again from memory."""
    heads, Lq, L = 10, 1024, 4096
    g = torch.Generator(device=DEV).manual_seed(73)
    q, k, v = (torch.randn(1, n, heads * 64, generator=g, device=DEV) for n in (Lq, L, L))
    k, vt = k.to(torch.bfloat16), v.to(torch.bfloat16).transpose(1, 2).contiguous()

    def best(std):
        qs, times = (std * q).to(torch.bfloat16), []
        out = [df.attn_stale_vt(qs, k, vt, heads, L) for _ in range(3)]
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            out = [df.attn_stale_vt(qs, k, vt, heads, L) for _ in range(20)]
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / len(out))
        return min(times)

    flat, peaked = best(0.25), best(8.0)
    say("attention of flat scores %.1f us, of peaked scores %.1f us" % (1e3 * flat, 1e3 * peaked))
    assert peaked < 1.4 * flat
