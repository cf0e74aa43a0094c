"""Timed cases of the diff encoder: whole groups of pictures -- a reference
frame and the diff frames that follow it -- through SparseTemNet.

A case names a net, its input size and dtype, the schedule its frames take
("chunk": all diff frames in one encode_chunk call; "frame": one encode_diff
call each, as a live stream does; "reference": the dense pass alone), how
many frames the group has, which share of the sites changes from one frame
to the next, the truncation threshold and the creation option.

Nets (weights random, drawn on the device from the seed):
  toy     3x3 conv 16 -> 16, ReLU, 1x1 conv 16 -> 32: the smallest encoder
  crnn    CRNN-VGG text-line encoder: seven 3x3 convs, four max-pools
  resnet  ResNet-50: 7x7/2 stem, overlapping pool, bottleneck blocks
  b0      EfficientNet-B0: depthwise convs, SiLU, squeeze-excitation
"""

import functools
import math
import random
from types import SimpleNamespace

import numpy as np
import torch
import torch.nn.functional as F

from paper_2410_20790_amd import SparseTemNet

NONE, RELU, SILU = 0, 1, 2
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ESIZE = {"f32": 4, "f16": 2, "bf16": 2}
CHANNELS = {"toy": 16, "crnn": 1, "resnet": 3, "b0": 3}


def _case(name, net, dtype, batch, h, w, schedule, frames, change, thr,
          option="none"):
    return dict(name=name, net=net, dtype=dtype, batch=batch, h=h, w=w,
                schedule=schedule, frames=frames, change=change, thr=thr,
                option=option)


def listed():
    return [
        # the smallest call: two layers on a small frame, all launch latency
        _case("toy_chunk", "toy", "f32", 1, 64, 64, "chunk", 4, 0.10, 0.0),
        # a text line scrolling through a fixed window, as a recogniser
        # reads it: in chunks of 16, and live, frame by frame
        _case("crnn_chunk", "crnn", "f32", 1, 32, 128, "chunk", 16, 0.055,
              0.02),
        _case("crnn_live", "crnn", "f32", 3, 32, 128, "frame", 6, 0.055,
              0.02),
        # driving video on ResNet-50, exact (threshold 0): whole chunks, the
        # dense reference pass alone, and live, frame by frame
        _case("resnet_chunk", "resnet", "bf16", 1, 1024, 2048, "chunk", 10,
              0.10, 0.0),
        _case("resnet_reference", "resnet", "bf16", 1, 1024, 2048,
              "reference", 1, 0.0, 0.0),
        _case("resnet_live", "resnet", "bf16", 1, 1024, 2048, "frame", 3,
              0.10, 0.0),
        # an odd-sized camera at the lossy setting
        _case("resnet_ragged", "resnet", "f16", 1, 375, 621, "chunk", 8,
              0.20, 0.02),
        # residual carry, the accuracy option of the lossy setting
        _case("resnet_carry", "resnet", "bf16", 1, 512, 1024, "chunk", 6,
              0.10, 0.02, "carry"),
        # a detector backbone on one camera: chunks, and live
        _case("b0_chunk", "b0", "f16", 1, 512, 512, "chunk", 8, 0.08, 0.05),
        _case("b0_live", "b0", "f16", 1, 512, 512, "frame", 4, 0.08, 0.05),
        # 32 cameras as the images of one net
        _case("b0_cameras", "b0", "bf16", 32, 256, 256, "chunk", 8, 0.15,
              0.05),
        # the memory-saving options together, on an odd size, exact
        _case("b0_frozen", "b0", "bf16", 2, 301, 427, "chunk", 5, 0.05, 0.0,
              "frozen_bf16state"),
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    net = rng.choice(["toy", "crnn", "resnet", "resnet", "b0", "b0"])
    schedule = rng.choice(["chunk", "chunk", "frame", "reference"])
    thr = rng.choice([0.0, 0.02, 0.05])
    change = round(rng.uniform(0.02, 0.30), 3)
    option = "none"
    if net == "toy":
        dtype = rng.choice(["f32", "f16"])
        batch, frames = rng.randint(1, 4), rng.randint(2, 8)
        h, w = _between(rng, 16, 256), _between(rng, 16, 256)
    elif net == "crnn":
        dtype = rng.choice(["f32", "f16"])
        batch, frames = rng.randint(1, 4), rng.randint(2, 16)
        h, w = 32, _between(rng, 64, 512)
    elif net == "resnet":
        dtype = rng.choice(["f16", "bf16", "bf16", "f32"])
        option = rng.choice(["none", "none", "carry"])
        batch, frames = rng.randint(1, 2), rng.randint(2, 10)
        h = _between(rng, 64, 1024)
        w = _between(rng, h, 2 * h)
    else:
        dtype = rng.choice(["f16", "bf16", "f32"])
        option = rng.choice(["none", "none", "carry", "frozen",
                             "frozen_bf16state"])
        h = _between(rng, 96, 512)
        w = rng.randint(h * 3 // 4, h)
        batch, frames = _between(rng, 1, 32), rng.randint(2, 8)
    if schedule == "reference":
        frames, change, thr = 1, 0.0, 0.0
    elif schedule == "chunk":
        frames = max(frames, 3)
    elif net in ("resnet", "b0"):
        frames = min(frames, 4)
    if net in ("resnet", "b0"):
        # no more work than the largest listed case: weigh the sites by what
        # the options cost, and make the images smaller if need be
        most = 1024 * 2048 * (3.0 if net == "resnet" else 2.0)
        weight = 1 + (frames - 1) * (0.1 + 2 * change)
        if net == "b0" and thr == 0 and option in ("none", "carry"):
            weight *= 2
        weight *= {"f32": 4, "f16": 1, "bf16": 1}[dtype]
        weight *= 2.5 if option == "carry" else 1
        sites = batch * h * w * weight
        if sites > most:
            batch = max(1, min(batch, int(batch * most / sites)))
            shrink = min(1.0, (most / (batch * h * w * weight)) ** 0.5)
            h, w = max(48, int(h * shrink)), max(48, int(w * shrink))
    c = _case("", net, dtype, batch, h, w, schedule, frames, change, thr,
              option)
    del c["name"]
    return c


# ---- nets

def _conv(src, cin, cout, k, s=1, act=RELU, groups=1, res=-2, pool=None,
          se_mid=0, gain=1.0):
    pk, ps, pp = pool or ((0, 0), (0, 0), (0, 0))
    return SimpleNamespace(src=src, residual_src=res, c_in=cin, c_out=cout,
                           groups=groups, k=(k, k), s=(s, s),
                           p=(k // 2, k // 2), act=act, pool_k=pk, pool_s=ps,
                           pool_p=pp, se_mid=se_mid, gain=gain)


def _toy():
    return [_conv(-1, 16, 16, 3), _conv(0, 16, 32, 1, act=NONE)]


def _crnn():
    pools = {0: (2, 2), 1: (2, 2), 3: (2, 1), 5: (2, 1)}
    layers, cin = [], 1
    for i, c in enumerate([64, 128, 256, 256, 512, 512, 512]):
        pool = (pools[i], pools[i], (0, 0)) if i in pools else None
        layers.append(_conv(i - 1, cin, c, 3, pool=pool))
        cin = c
    return layers


def _resnet():
    layers = [_conv(-1, 3, 64, 7, 2, pool=((3, 3), (2, 2), (1, 1)))]
    prev, cin = 0, 64
    for stage, (blocks, width) in enumerate(zip((3, 4, 6, 3),
                                                (64, 128, 256, 512))):
        for b in range(blocks):
            s = 2 if stage and not b else 1
            block_in, cout = prev, 4 * width
            layers.append(_conv(block_in, cin, width, 1))
            layers.append(_conv(len(layers) - 1, width, width, 3, s))
            mid = res = len(layers) - 1
            if b == 0:
                layers.append(_conv(block_in, cin, cout, 1, s, act=NONE))
                res = len(layers) - 1
            else:
                res = block_in
            layers.append(_conv(mid, width, cout, 1, res=res, gain=0.2))
            prev, cin = len(layers) - 1, cout
    return layers


def _b0():
    layers = [_conv(-1, 3, 32, 3, 2, act=SILU)]
    prev, cin = 0, 32
    for t, k, s, c, n in [(1, 3, 1, 16, 1), (6, 3, 2, 24, 2),
                          (6, 5, 2, 40, 2), (6, 3, 2, 80, 3),
                          (6, 5, 1, 112, 3), (6, 5, 2, 192, 4),
                          (6, 3, 1, 320, 1)]:
        for b in range(n):
            s = s if b == 0 else 1
            block_in, mid = prev, cin * t
            src = block_in
            if t > 1:
                layers.append(_conv(src, cin, mid, 1, act=SILU))
                src = len(layers) - 1
            layers.append(_conv(src, mid, mid, k, s, act=SILU, groups=mid,
                                se_mid=max(1, cin // 4)))
            keep = s == 1 and cin == c
            layers.append(_conv(len(layers) - 1, mid, c, 1, act=NONE,
                                res=block_in if keep else -2, gain=0.5))
            prev, cin = len(layers) - 1, c
    return layers


NETS = {"toy": _toy, "crnn": _crnn, "resnet": _resnet, "b0": _b0}


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _generator(seed, stream):
    g = torch.Generator(device=_device())
    g.manual_seed((int(seed) * 1000003 + stream) % (1 << 62))
    return g


def _weights(case, seed):
    """The case's layers with weights of its storage dtype (host arrays)."""
    g = _generator(seed, 1)
    dt = TORCH[case["dtype"]]

    def normal(shape, std, mean=0.0):
        x = torch.randn(shape, generator=g, device=g.device) * std + mean
        return x.to(dt).to(torch.float32).cpu().numpy()

    layers = NETS[case["net"]]()
    for L in layers:
        cg = L.c_in // L.groups
        std = L.gain * math.sqrt(2.0 / (cg * L.k[0] * L.k[1]))
        bias = 0.02
        if case["net"] == "toy":
            std = bias = 0.1
        L.weight = normal((L.c_out, cg) + L.k, std)
        L.bias = normal((L.c_out,), bias)
        if L.se_mid:
            L.se_w1 = normal((L.se_mid, L.c_out), math.sqrt(2.0 / L.c_out))
            L.se_b1 = normal((L.se_mid,), 0.02)
            L.se_w2 = normal((L.c_out, L.se_mid), math.sqrt(1.0 / L.se_mid))
            L.se_b2 = normal((L.c_out,), 0.2, 1.0)
    return layers


# ---- frames

def _changed(case, seed):
    """Which sites each diff frame re-draws: bool [frames - 1, N, H, W].
    Text lines: a band of columns that moves on from frame to frame;
    elsewhere: the union of rectangles (the sides follow the frame's size),
    as moving objects leave it."""
    n, h, w = case["batch"], case["h"], case["w"]
    rng = random.Random(int(seed) * 7919 + 17)
    out = np.zeros((case["frames"] - 1, n, h, w), bool)
    for i in range(n):
        at = rng.randrange(w)
        for t in range(case["frames"] - 1):
            m = out[t, i]
            if case["net"] == "crnn":
                band = max(1, round(case["change"] * w))
                m[:, [(at + j) % w for j in range(band)]] = True
                at = (at + band) % w
                continue
            lo, hi = max(4, h // 32), max(5, h // 4)
            if case["net"] == "toy":
                lo = hi = 8
            while m.mean() < case["change"]:
                a, b = rng.randint(lo, hi), rng.randint(lo, hi)
                y, x = rng.randrange(1 - a // 2, h), rng.randrange(
                    1 - b // 2, w)
                m[max(0, y):y + a, max(0, x):x + b] = True
    return out


def _frames(case, seed):
    """[frames, N, H, W, C] in the storage dtype, values in [0, 1]: smooth
    content plus texture; a re-drawn site changes in every channel."""
    n, h, w = case["batch"], case["h"], case["w"]
    c = CHANNELS[case["net"]]
    g = _generator(seed, 2)
    dev, dt = g.device, TORCH[case["dtype"]]

    def noise(*shape):
        return torch.rand(shape, generator=g, device=dev)

    if case["net"] == "crnn":  # dark strokes on a light line

        def fresh():
            f = torch.where(noise(n, h, w, 1) < 0.3, 0.1, 0.85)
            f[:, :h // 6] = 0.85
            f[:, h - h // 6:] = 0.85
            return f
        x = fresh()
    elif case["net"] == "toy":
        def fresh():
            return noise(n, h, w, c)
        x = fresh()
    else:
        x = torch.zeros((n, c, h, w), device=dev)
        for o, amp in enumerate((0.5, 0.25, 0.15, 0.1)):
            low = noise(n, c, max(2, (h << o) // 64), max(2, (w << o) // 64))
            x += amp * F.interpolate(low, size=(h, w), mode="bilinear",
                                     align_corners=False)
        x = x.permute(0, 2, 3, 1).contiguous()
        base = x.clone()

        def fresh():
            return 0.5 * base + 0.5 * noise(n, h, w, c)
    out = torch.empty((case["frames"], n, h, w, c), dtype=dt, device=dev)
    out[0] = x.to(dt)
    if case["frames"] > 1:
        changed = torch.from_numpy(_changed(case, seed)).to(dev)
        for t in range(1, case["frames"]):
            new = fresh().to(dt)
            same = new == out[t - 1]
            if case["net"] == "crnn":  # a re-drawn stroke really moves
                new = torch.where(same, torch.where(new > 0.5, 0.1, 0.85).to(
                    dt), new)
            else:
                new = torch.where(same, (0.99 - new.float() * 0.5).to(dt),
                                  new)
            out[t] = torch.where(changed[t - 1][..., None], new, out[t - 1])
    return out


# ---- the timed path

def prepare(case, seed):
    diffs = case["frames"] - 1
    opt = case["option"]
    layers = _weights(case, seed)
    net = SparseTemNet(
        layers, case["batch"], case["h"], case["w"], CHANNELS[case["net"]],
        case["dtype"],
        max_frames=diffs if case["schedule"] == "chunk" else 1,
        carry=opt == "carry", frozen_se=opt.startswith("frozen"),
        bf16_state=opt == "frozen_bf16state")
    return {"schedule": case["schedule"], "net": net,
            "frames": _frames(case, seed),
            "thr": [case["thr"]] * (len(layers) + 1),
            "ref": net.new_output(),
            "diff": torch.empty((diffs,) + tuple(net.out_shape),
                                dtype=torch.float32, device=net.device)}


def run(state):
    net, frames = state["net"], state["frames"]
    net.encode_reference(frames[0], state["ref"])
    if state["schedule"] == "reference":
        return {"ref": state["ref"]}
    if state["schedule"] == "chunk":
        net.encode_chunk(frames[1:], state["thr"], state["diff"])
    else:
        for t in range(1, frames.shape[0]):
            net.encode_diff(frames[t], state["thr"], state["diff"][t - 1])
    return {"ref": state["ref"], "diff": state["diff"]}


def _out_hw(L, h, w):
    ho = (h + 2 * L.p[0] - L.k[0]) // L.s[0] + 1
    wo = (w + 2 * L.p[1] - L.k[1]) // L.s[1] + 1
    if not L.pool_k[0]:
        return ho, wo, ho, wo
    return (ho, wo, (ho + 2 * L.pool_p[0] - L.pool_k[0]) // L.pool_s[0] + 1,
            (wo + 2 * L.pool_p[1] - L.pool_k[1]) // L.pool_s[1] + 1)


@functools.lru_cache(maxsize=64)
def _work(items):
    """The reference frame's dense products; for the diff frames those of
    the changed sites: with threshold 0 as far as the windows carry a change
    (exact squeeze-excitation: everywhere), with a larger one the re-drawn
    sites alone (what a window carries past them is mostly dropped).  Bytes:
    frames, weights and outputs, each layer's input read and its state
    written (and, in a diff frame, read) at the sites counted."""
    case = dict(items)
    es = ESIZE[case["dtype"]]
    layers = NETS[case["net"]]()
    n, diffs = case["batch"], case["frames"] - 1
    exact = case["thr"] == 0
    sb = 2 if case["option"] == "frozen_bf16state" else 4
    shape = {-1: (case["h"], case["w"])}
    act, own = {}, {}
    if diffs:
        m = torch.from_numpy(_changed(case, 0)).reshape(
            diffs * n, 1, case["h"], case["w"]).to(_device(), torch.float32)
        act[-1] = m
        own[-1] = float(m.sum())
    flops = 0.0
    nbytes = n * case["frames"] * case["h"] * case["w"] * CHANNELS[
        case["net"]] * es
    for i, L in enumerate(layers):
        hi, wi = shape[L.src]
        ho, wo, hp, wp = _out_hw(L, hi, wi)
        shape[i] = (hp, wp)
        per_pair = 2.0 * (L.c_in // L.groups) * L.c_out
        kk = L.k[0] * L.k[1]
        nbytes += kk * (L.c_in // L.groups) * L.c_out * es
        flops += n * ho * wo * kk * per_pair
        state = L.act != NONE or L.pool_k[0] > 0 or i == len(layers) - 1
        nbytes += n * (hi * wi * L.c_in * es + state * ho * wo * L.c_out * sb)
        if diffs:
            m = act[L.src]
            flops += own[L.src] * kk / (L.s[0] * L.s[1]) * per_pair
            if exact:
                m = F.max_pool2d(m, L.k, L.s, L.p)
            elif L.s[0] > 1:
                m = F.max_pool2d(m, L.s, L.s, ceil_mode=True)[..., :ho, :wo]
            if exact and L.residual_src != -2:
                m = torch.maximum(m, act[L.residual_src])
            sites = float(m.sum())
            nbytes += own[L.src] * L.c_in * es
            nbytes += state * 2 * sites * L.c_out * sb
            if L.pool_k[0]:
                k = L.pool_k if exact else L.pool_s
                p = L.pool_p if exact else (0, 0)
                m = F.max_pool2d(m, k, L.pool_s, p,
                                 ceil_mode=not exact)[..., :hp, :wp]
            if exact and L.se_mid and case["option"] in ("none", "carry"):
                m = torch.ones_like(m)
            act[i], own[i] = m, float(m.sum())
    hl, wl = shape[len(layers) - 1]
    nbytes += case["frames"] * n * hl * wl * layers[-1].c_out * 4
    return {"bytes": float(nbytes), "flops": float(flops)}


def work(case):
    return dict(_work(tuple(sorted((k, v) for k, v in case.items()
                                   if k != "name"))))


def tolerance(case):
    """About four times what the sums in another order give: chunks against
    frame-by-frame encoding differ by up to 4.3e-7 (f32), 2.9e-4 (f16) and
    7.8e-4 (bf16) with the reference frame's sums the same, and the half
    precision nets are 9e-4 and 7e-3 from the f64 result.  With a threshold
    above 0 a row whose delta equals it but for the rounding may be kept on
    one side only, a difference of the threshold's size at that row."""
    if case["thr"] == 0:
        return {"rel": {"f32": 3e-6, "f16": 2e-3, "bf16": 1e-2}[
            case["dtype"]]}
    return {"rel": {"f32": 1e-4, "f16": 4e-3, "bf16": 1.5e-2}[case["dtype"]]}


@torch.no_grad()
def exact(case, seed):
    """Dense f64 forward of every frame: with threshold 0 (and, by the
    convolution's linearity, only then) the diff frames' result too."""
    dev = _device()
    layers = _weights(case, seed)
    frames = _frames(case, seed).to(torch.float64)

    def t64(x):
        return torch.from_numpy(x).to(dev, torch.float64)

    params = [[t64(L.weight), t64(L.bias)] + (
        [t64(x) for x in (L.se_w1, L.se_b1, L.se_w2, L.se_b2)]
        if L.se_mid else []) for L in layers]
    last = {}
    for i, L in enumerate(layers):
        last[L.src] = last[L.residual_src] = i
    gates = {}

    def dense(x, first):
        vals = {-1: x.permute(0, 3, 1, 2).contiguous()}
        for i, (L, p) in enumerate(zip(layers, params)):
            v = F.conv2d(vals[L.src], p[0], p[1], L.s, L.p, 1, L.groups)
            if L.residual_src != -2:
                v += vals[L.residual_src]
            v = F.relu(v) if L.act == RELU else (
                F.silu(v) if L.act == SILU else v)
            if L.pool_k[0]:
                v = F.max_pool2d(v, L.pool_k, L.pool_s, L.pool_p)
            if L.se_mid:
                if first or not case["option"].startswith("frozen"):
                    z = F.silu(v.mean((2, 3)) @ p[2].T + p[3])
                    gates[i] = torch.sigmoid(z @ p[4].T + p[5])
                v = v * gates[i][:, :, None, None]
            vals[i] = v
            for s in [s for s in vals if last.get(s, 1 << 30) <= i]:
                del vals[s]
        return vals[len(layers) - 1].permute(0, 2, 3, 1).contiguous()

    out = {"ref": dense(frames[0], True)}
    if case["schedule"] != "reference":
        out["diff"] = None
        if case["thr"] == 0:
            out["diff"] = torch.stack([dense(f, False) for f in frames[1:]])
    return out
