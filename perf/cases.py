"""Performance cases of the displaced-patch UNet on one MI355X: what a user of the library has it do.

A user keeps a `PatchUNet` (weights laid out once, workspace, stale state) and calls `step` for every denoising step of
their patch, or lets `sample_patch` run the whole Euler loop; somebody who builds their own network calls the single
operations (GroupNorm with stale sums, halo convolution, displaced attention, linear layer, refresh).  The listed cases
take both from the smallest problem to the largest, `draw` gives further sizes of the same ranges.

Kinds of cases
  block   float32 GroupNorm -> halo convolution -> displaced self-attention of a small block
  layer   bf16 displaced self-attention layer: three projections, attention on spliced keys / values, output projection
  stage   GroupNorm + SiLU -> halo convolution (stride 1 or 2), bf16 or float32, horizontal or vertical strips
  norm    GroupNorm + SiLU of a patch, then the refresh of the full stale buffer with the result
  step    one UNet step: DISPLACED + refresh of one patch, or the synchronous FULL step
  loop    `PatchUNet.sample_patch`: one synchronous step, then displaced ones, with the sampler's updates
"""
import math

import torch

import paper_2402_19481_amd as df
from df_inputs import unet_table as ut

DEV = "cuda:0"
G = 32          # GroupNorm groups of every bf16 configuration
_stream = None  # the program's one working stream (steps replay as a HIP graph, which the default stream does not allow)


def _work_stream():
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def listed():
    return [
        # the tiny float32 configuration: three launches of a few microseconds, nothing but latency
        dict(name="block_16x16x32_f32", kind="block", H=16, W=16, C=32, N=2),
        # one self-attention layer of the middle level of a 1024x1024 image cut into 4 patches
        dict(name="layer_1024_of_4096", kind="layer", H=64, W=64, C=640, N=4, B=1, axis="rows"),
        # the residual block's first half at the top level of a 1024x1024 image cut into 4 patches
        dict(name="stage_128x128x320", kind="stage", H=128, W=128, C=320, Cout=320, N=4, B=1, stride=1, axis="rows",
             dtype="bf16"),
        # the largest GroupNorm of a 2048x2048 image (concatenated skip, 31 MB), and the refresh of its stale buffer
        dict(name="norm_64x256x960", kind="norm", R=64, W=256, C=960, N=4, B=1),
        # a 512x512 image over 4 patches: few tokens per patch, the weights are most of what has to move
        dict(name="step_512", kind="step", H=64, W=64, N=4, B=1, patch=1, mode="displaced", axis="rows"),
        # a 1024x1024 image over 8 patches with both classifier-free-guidance branches in the batch
        dict(name="step_1024_guided", kind="step", H=128, W=128, N=8, B=2, patch=3, mode="displaced", axis="rows"),
        # a non-square image over 2 patches: ragged token counts at every level
        dict(name="step_832x1216", kind="step", H=104, W=152, N=2, B=1, patch=1, mode="displaced", axis="rows"),
        # the benchmark's step: 1280x1920 over 8 patches
        dict(name="step_1280x1920", kind="step", H=160, W=240, N=8, B=1, patch=3, mode="displaced", axis="rows"),
        # 2048x2048 over 4 vertical strips
        dict(name="step_2048_strips", kind="step", H=256, W=256, N=4, B=1, patch=1, mode="displaced", axis="cols"),
        # 3840x3840 over 8 patches, the largest image
        dict(name="step_3840", kind="step", H=480, W=480, N=8, B=1, patch=3, mode="displaced", axis="rows"),
        # the synchronous first step of a 1024x1024 image
        dict(name="full_1024", kind="step", H=128, W=128, N=4, B=1, patch=0, mode="full", axis="rows"),
        # the sampling loop of one of two devices at 768x768: a synchronous step, then displaced ones
        dict(name="loop_768", kind="loop", H=96, W=96, N=2, B=1, patch=0, steps=5),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _cfg(c):
    return ut.UNetCfg(H=c["H"], W=c["W"], N=c["N"], **ut.SDXL)


def _tflop(c):
    if c.get("axis") == "cols":      # the count knows horizontal strips: the same work on the transposed image
        c = dict(c, H=c["W"], W=c["H"])
    return 2e-12 * c["B"] * ut.count_macs(_cfg(c), 1 if c.get("mode") == "full" else None)["total"]


def draw(rng):
    kind = rng.choice(["block", "layer", "layer", "stage", "stage", "norm", "norm", "step", "step", "step", "step", "full",
                       "loop"])
    if kind == "block":
        N = rng.choice([1, 2, 4])
        return dict(kind=kind, H=N * int(_log(rng, 4, 24)), W=int(_log(rng, 5, 48)), C=rng.choice([32, 64]), N=N)
    if kind == "layer":
        N = rng.choice([2, 4, 8])
        axis = rng.choice(["rows", "rows", "cols"])
        other, part = int(_log(rng, 10, 160)), int(_log(rng, 3, 40))
        H, W = (part * N, other) if axis == "rows" else (other, part * N)
        return dict(kind=kind, H=H, W=W, C=rng.choice([320, 640, 1280]), N=N, B=rng.choice([1, 1, 2]), axis=axis)
    if kind == "stage":
        N = rng.choice([2, 4, 8])
        axis = rng.choice(["rows", "rows", "cols"])
        f32 = rng.random() < 0.2
        stride = rng.choice([1, 1, 1, 2])
        step = 2 if stride == 2 else 1
        part = step * int(_log(rng, 3, 40 if not f32 else 12))
        other = step * int(_log(rng, 8, 120 if not f32 else 24))
        H, W = (part * N, other) if axis == "rows" else (other, part * N)
        C = rng.choice([32, 64]) if f32 else rng.choice([320, 640, 960, 1280, 1920])
        Cout = C if f32 or stride == 2 else rng.choice([320, 640, 1280])
        return dict(kind=kind, H=H, W=W, C=C, Cout=Cout, N=N, B=rng.choice([1, 1, 2]), stride=stride, axis=axis,
                    dtype="f32" if f32 else "bf16")
    if kind == "norm":
        return dict(kind=kind, R=int(_log(rng, 3, 96)), W=int(_log(rng, 12, 300)), C=rng.choice([320, 640, 960, 1280, 1920, 2560]),
                    N=rng.choice([2, 4, 8]), B=rng.choice([1, 1, 2]))
    while True:
        if kind == "step":
            N = rng.choice([2, 4, 8])
            part, other = 4 * int(_log(rng, 2, 17)), 4 * int(_log(rng, 10, 100))
            axis = rng.choice(["rows", "rows", "rows", "cols"])
            H, W = (part * N, other) if axis == "rows" else (other, part * N)
            c = dict(kind="step", H=H, W=W, N=N, B=rng.choice([1, 1, 2]), patch=rng.randrange(N), mode="displaced", axis=axis)
            most = 15.0
        elif kind == "full":
            c = dict(kind="step", H=8 * int(_log(rng, 7, 22)), W=4 * int(_log(rng, 14, 44)), N=2, B=rng.choice([1, 1, 2]), patch=0,
                     mode="full", axis="rows")
            most = 18.0
        else:
            N = rng.choice([2, 4])
            c = dict(kind="loop", H=4 * N * int(_log(rng, 4, 10)), W=4 * int(_log(rng, 14, 36)), N=N, B=1, patch=rng.randrange(N),
                     steps=rng.randrange(3, 7))
            most = 4.0
        # the stale state and the synchronous step that fills it stay within what the largest listed case needs
        if 0.4 <= _tflop(c) <= most and c["H"] * c["W"] * c["B"] <= 480 * 480:
            return c


# ---- inputs -------------------------------------------------------------------------------------------------------------

class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed))

    def f32(self, *shape, std=1.0, mean=0.0):
        return torch.randn(*shape, generator=self.g, device=DEV).mul_(std).add_(mean)

    def typed(self, dtype, *shape, std=1.0):
        return self.f32(*shape, std=std).to(dtype)


def _weights(r, specs):
    """Random-init parameters: matrices N(0, 1/fan_in) in bf16, biases 0.02, norm scale 1 + 0.1, shift 0.1 N(0,1)."""
    out = []
    for name, shape in specs:
        if name.endswith(".w"):
            out.append(r.typed(torch.bfloat16, *shape, std=math.prod(shape[1:]) ** -0.5))
        elif name.endswith(".g"):
            out.append(r.f32(*shape, std=0.1, mean=1.0))
        else:
            out.append(r.f32(*shape, std=0.1 if name.endswith(".beta") else 0.02))
    return out


def _patch_stats(r, x_full, groups, N, dim):
    """Per-patch (sum, sum of squares) of the previous step's activation, [N, B, groups, 2]."""
    parts = torch.stack([p.float().reshape(p.shape[0], -1, groups, p.shape[3] // groups) for p in x_full.chunk(N, dim)])
    return torch.stack([parts.sum((2, 4)), parts.square().sum((2, 4))], -1).contiguous()


def _fresh(r, stale, p, N, dim, dtype):
    """This step's activation of patch p: the previous step's plus the usual difference between two steps."""
    part = stale.chunk(N, dim)[p].float()
    return (part + r.f32(*part.shape, std=0.02)).to(dtype).contiguous()


def _views(net):
    """The stale state as tensors: runs of neighbouring bf16 buffers (boundary rows, keys, values) and of GroupNorm sums."""
    base, runs = net.stale.data_ptr(), []
    for name in net.stale_names():
        v = net.stale_view(name)
        lo, hi, dt = v.data_ptr() - base, v.data_ptr() - base + v.numel(), torch.float32 if name.endswith(".stats") else torch.bfloat16
        if runs and runs[-1][2] == dt and 0 <= lo - runs[-1][1] < 256:
            runs[-1][1] = hi
        else:
            runs.append([lo, hi, dt])
    return [net.stale[lo:hi].view(dt) for lo, hi, dt in runs]


def prepare(case, seed):
    r, c = _Rand(seed), case
    k = c["kind"]
    s = dict(case=c, stream=_work_stream())
    if k == "block":
        H, W, C, N = c["H"], c["W"], c["C"], c["N"]
        p = N - 1
        stale = r.f32(1, H, W, C)
        s.update(p=p, stale=stale, x=_fresh(r, stale, p, N, 1, torch.float32), stats=_patch_stats(r, stale, 8, N, 1),
                 gamma=r.f32(C, std=0.1, mean=1.0), beta=r.f32(C, std=0.1), w=r.f32(C, 3, 3, C, std=(9 * C) ** -0.5),
                 b=r.f32(C, std=0.02), ks=r.f32(1, H * W, C), vs=r.f32(1, H * W, C))
    elif k == "layer":
        H, W, C, N, B = c["H"], c["W"], c["C"], c["N"], c["B"]
        bf, L = torch.bfloat16, H * W
        s.update(p=1, x=r.typed(bf, B * L // N, C), w=[r.typed(bf, C, C, std=C ** -0.5) for _ in range(4)], b=r.f32(C, std=0.02),
                 ks=r.typed(bf, B, L, C), vs=r.typed(bf, B, L, C))
    elif k == "stage":
        H, W, C, N, B = c["H"], c["W"], c["C"], c["N"], c["B"]
        dt, dim, p = torch.float32 if c["dtype"] == "f32" else torch.bfloat16, 1 if c["axis"] == "rows" else 2, 1
        stale = r.typed(dt, B, H, W, C)
        s.update(p=p, stale=stale, x=_fresh(r, stale, p, N, dim, dt), stats=_patch_stats(r, stale, 8 if C < 320 else G, N, dim),
                 gamma=r.f32(C, std=0.1, mean=1.0), beta=r.f32(C, std=0.1),
                 w=r.typed(dt, c["Cout"], 3, 3, C, std=(2.0 / (9 * C)) ** 0.5), b=r.f32(c["Cout"], std=0.02))
    elif k == "norm":
        R, W, C, N, B = c["R"], c["W"], c["C"], c["N"], c["B"]
        stale = r.typed(torch.bfloat16, B, R * N, W, C)
        s.update(p=1, stale=stale, x=_fresh(r, stale, 1, N, 1, torch.bfloat16), stats=_patch_stats(r, stale, G, N, 1),
                 gamma=r.f32(C, std=0.1, mean=1.0), beta=r.f32(C, std=0.1))
    else:
        cfg, B = _cfg(c), c["B"]
        cols = c.get("axis") == "cols"
        axis = df.SPLIT_COLS if cols else df.SPLIT_ROWS
        net = df.PatchUNet(cfg, _weights(r, df.unet_weight_specs(df.make_cfg(cfg, B, axis))), B=B, split_axis=axis)
        emb, text = r.f32(B, cfg.emb_dim), r.typed(torch.bfloat16, B, cfg.text_len, cfg.text_dim)
        x_prev = r.f32(B, cfg.H, cfg.W, cfg.in_ch)
        s.update(net=net, emb=emb, text=text)
        if k == "loop":
            n = c["steps"]
            s["sigmas"] = [14.6 * (0.03 / 14.6) ** (i / n) for i in range(n + 1)]
            s["x0"] = x_prev * s["sigmas"][0]
            s["state"] = [v for v in _views(net) if v.dtype == torch.bfloat16]
            return s
        x = x_prev + r.f32(*x_prev.shape, std=0.02)
        if c["mode"] == "displaced":
            # the previous, synchronous step left the stale state
            s["stream"].wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s["stream"]):
                net.step(x_prev, emb, text, mode=df.MODE_FULL, out=x_prev.clone())
            torch.cuda.current_stream().wait_stream(s["stream"])
            x = x.chunk(c["N"], 2 if cols else 1)[c["patch"]].contiguous()
        s.update(x=x, eps=torch.empty_like(x), state=_views(net))
    return s


def run(s):
    c = s["case"]
    k, N = c["kind"], c.get("N")
    with torch.cuda.stream(s["stream"]):
        if k == "step":
            mode = df.MODE_FULL if c["mode"] == "full" else df.MODE_DISPLACED
            s["net"].step(s["x"], s["emb"], s["text"], patch_idx=c["patch"], mode=mode, refresh=True, out=s["eps"])
            return [s["eps"], s["state"]]
        if k == "loop":
            x = s["x0"].clone()
            return [s["net"].sample_patch(x, s["emb"], s["text"], s["sigmas"], c["patch"]), x, s["state"]]
        if k == "layer":
            B, C, heads, L = c["B"], c["C"], c["C"] // 64, c["H"] * c["W"]
            q, kf, vf = (df.linear(s["x"], w).view(B, L // N, C) for w in s["w"][:3])
            if c["axis"] == "rows":
                o = df.attn_displaced(q, kf, vf, s["ks"], s["vs"], heads, s["p"], N)
            else:
                o = df.attn_displaced_cols(q, kf, vf, s["ks"], s["vs"], heads, c["H"], c["W"], s["p"], N)
            return [df.linear(o.view(-1, C), s["w"][3], bias=s["b"]), kf, vf]
        groups = 8 if c["C"] < 320 else G
        y, stats = df.groupnorm_stale(s["x"], s["stats"], s["gamma"], s["beta"], groups, s["p"], N, fuse_silu=k != "block")
        if k == "norm":
            return [y, stats, df.buffer_refresh(s["stale"], y, s["p"], N)]
        if k == "block":
            z = df.conv3x3_halo(y, s["stale"], s["w"], s["b"], s["p"], N)
            t = z.view(1, -1, c["C"])
            return [y, stats, z, df.attn_displaced(t, t, t, s["ks"], s["vs"], 1 if c["C"] == 32 else c["C"] // 64, s["p"], N)]
        conv = df.conv3x3_halo if c["axis"] == "rows" else df.conv3x3_halo_cols
        return [y, stats, conv(y, s["stale"], s["w"], s["b"], s["p"], N, stride=c["stride"], act=1)]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------

def _unet_work(c):
    """Weights once, keys / values of every self-attention once (the patch's own are written, the others' read)."""
    cfg = _cfg(c)
    by = 2.0 * ut.num_params(cfg) + 8.0 * c["B"] * cfg.H * cfg.W * cfg.in_ch / (1 if c.get("mode") == "full" else cfg.N)
    for b in ut.blocks(cfg):
        if b[0] == "xf":
            h, w = cfg.level_hw(b[4])
            by += 4.0 * c["B"] * h * w * b[2] * b[3]
    return by, 1e12 * _tflop(c)


def work(c):
    k = c["kind"]
    if k == "step":
        by, fl = _unet_work(c)
    elif k == "loop":
        by, fl = _unet_work(dict(c, mode="full"))
        b1, f1 = _unet_work(c)
        by, fl = by + (c["steps"] - 1) * b1, fl + (c["steps"] - 1) * f1
    elif k == "layer":
        L, C, B = c["H"] * c["W"], c["C"], c["B"]
        M = B * L // c["N"]
        by, fl = 2.0 * (4 * M * C + 4 * C * C + 2 * B * L * C - 2 * M * C), 8.0 * M * C * C + 4.0 * M * L * C
    elif k == "norm":
        e = c["B"] * c["R"] * c["W"] * c["C"]
        by, fl = 2.0 * 3 * e, 10.0 * e
    else:
        px, C = c["H"] * c["W"] // c["N"] * c.get("B", 1), c["C"]
        sz, Cout, st = 2.0 if c.get("dtype") == "bf16" else 4.0, c.get("Cout", C), c.get("stride", 1)
        by = sz * (2 * px * C + px // st ** 2 * Cout + 9 * C * Cout)
        fl = 18.0 * px // st ** 2 * C * Cout
        if k == "block":
            by, fl = by + 4.0 * (px * C + 2 * (c["H"] * c["W"] - px) * C), fl + 4.0 * px * c["H"] * c["W"] * C
    return {"bytes": by, "flops": fl}


def tolerance(c):
    k = c["kind"]
    if k in ("step", "loop"):
        # seventy transformer blocks of bf16 operands in a row amplify the rounding of each: one correct implementation is
        # up to 1.6e-2 from the exact result, so two of them are up to sqrt(2) times that apart
        return {"rel": 2.5e-2, "max": 0.5}
    if k == "block" or c.get("dtype") == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2, "max": 0.1} if k == "layer" else {"rel": 5e-3, "max": 0.05}
