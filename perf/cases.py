"""Performance cases: what a program does with this framework, over the range it does it.

A case is one call (or one training step) through ``ReuseNet``: reuse steps of
one to a thousand streams, dense passes, occlusion sweeps, gradients and the
step that follows new weights, on the nets and frame sizes that the benchmark
and the tests use (Atari-like frames at full size, halved and quartered; two
and three 3x3 layers, stacked frames, a strided DQN-style trunk).  Frames are
sprite sequences: a static random background with constant squares that move a
few pixels per frame, so most pixels stay the same from frame to frame.

``exact`` evaluates the same function with plain torch in float64.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch
import torch.nn.functional as F

from paper_1909_05632_amd import ReuseNet

FRAMES = 6                 # frames of a sequence, walked back and forth
LR = 1e-3

# (frames stacked as input channels, layers as (cout, k, stride, pad))
NETS = {
    "conv20": (1, ((20, 3, 1, 1),)),
    "conv40-80": (1, ((40, 3, 1, 1), (80, 3, 1, 1))),
    "stack4-conv40-80": (4, ((40, 3, 1, 1), (80, 3, 1, 1))),
    "conv64-128-128": (1, ((64, 3, 1, 1), (128, 3, 1, 1), (128, 3, 1, 1))),
    "stack4-dqn": (4, ((32, 8, 4, 0), (64, 4, 2, 0), (64, 3, 1, 0))),
}


def _case(name, kind, net, n, h, w, *, n_out=6, act="f32", frame="f32", head="tiles", sprites=6, smin=4, smax=8,
          vmax=3, patch=8):
    c = dict(kind=kind, net=net, n=n, h=h, w=w, n_out=n_out, act=act, frame=frame, head=head, sprites=sprites,
             smin=smin, smax=smax, vmax=vmax, patch=patch)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One environment acting on quarter-size byte frames: latency of a single step.
        _case("step-1x53x40", "step", "conv40-80", 1, 53, 40, frame="u8", sprites=3, smax=4, vmax=2),
        # A rollout worker's batch: 256 environments on half-size frames.
        _case("step-256x105x80", "step", "conv40-80", 256, 105, 80),
        # The same with the last four frames as input channels, bytes from the emulator.
        _case("step-512x105x80-stack4", "step", "stack4-conv40-80", 512, 105, 80, frame="u8"),
        # A strided DQN-style trunk: small grids, most tiles dirty.
        _case("step-256x84x84-dqn", "step", "stack4-dqn", 256, 84, 84, sprites=5, smin=3, smax=6, vmax=2),
        # Serving a thousand full-size streams, about 1% of the pixels changing (the benchmark's workload).
        _case("step-1024x210x160", "step", "conv64-128-128", 1024, 210, 160, n_out=18, sprites=10, smin=6, vmax=2),
        # Full-size streams kept in bfloat16, about 6% changing, byte frames.
        _case("step-256x210x160-bf16", "step", "conv64-128-128", 256, 210, 160, n_out=18, act="bf16", frame="u8",
              sprites=26, smin=10, smax=14),
        # Priming full-size streams: the dense pass.
        _case("full-32x210x160", "full", "conv64-128-128", 32, 210, 160, n_out=18),
        # New weights between rollouts: the SGD step and the all-dirty step after it.
        _case("update-256x105x80", "update", "conv40-80", 256, 105, 80),
        # An occlusion map of one half-size frame: an 8x8 patch at 4096 places.
        _case("variants-4096x105x80", "variants", "conv40-80", 4096, 105, 80),
        # The same on a full-size frame and the deeper net, fewer places.
        _case("variants-1024x210x160", "variants", "conv64-128-128", 1024, 210, 160, n_out=18),
        # A REINFORCE step of the rollout batch: forward with reuse, logit gradient, backward.
        _case("train-256x105x80", "train", "conv40-80", 256, 105, 80),
        # The same for the deeper net on a small ragged batch.
        _case("train-24x106x92", "train", "conv64-128-128", 24, 106, 92, n_out=18),
    ]


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 1e14)


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng: random.Random):
    kind = rng.choice(["step", "step", "step", "full", "update", "variants", "train", "train"])
    nets = {"variants": ["conv40-80", "conv64-128-128"],
            "train": ["conv40-80", "stack4-conv40-80", "conv64-128-128"],
            "update": ["conv40-80", "stack4-conv40-80", "conv64-128-128"]}.get(kind, list(NETS))
    net = rng.choice(nets)
    act = "bf16" if kind in ("step", "full") and net == "conv64-128-128" and rng.random() < 0.4 else "f32"
    big = net == "conv64-128-128"
    smin = rng.randint(3, 10)
    case = _case(None, kind, net, 1, rng.randint(40, 210 if big else 120), 4 * rng.randint(10, 40 if big else 26),
                 n_out=rng.choice([4, 6, 18]), act=act, frame=rng.choice(["f32", "u8"]),
                 head="full" if kind != "variants" and rng.random() < 0.15 else "tiles",
                 sprites=rng.randint(2, 26 if big else 8), smin=smin, smax=smin + rng.randint(0, 4),
                 vmax=rng.randint(1, 3), patch=rng.randint(4, 8))
    case["n"] = {"variants": lambda: _log_int(rng, 64, 4096), "train": lambda: _log_int(rng, 4, 256)}.get(
        kind, lambda: _log_int(rng, 1, 512))()
    most = max(_cost(c) for c in listed() if c["kind"] == ("train" if kind == "train" else "step"))
    while case["n"] > 1 and (_cost(case) > most or case["n"] * case["h"] * case["w"] > 1 << 24):
        case["n"] -= case["n"] // 3 + 1
    case["n"] = max(1, case["n"])
    return case


# ---------------------------------------------------------------- geometry and work

def _layers(case):
    """(cin, cout, k, stride, pad, H, W of the output) per layer."""
    stack, convs = NETS[case["net"]]
    c, h, w, out = stack, case["h"], case["w"], []
    for cout, k, s, p in convs:
        h, w = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
        out.append((c, cout, k, s, p, h, w))
        c = cout
    return out


def _positions(case, n, seed):
    """Top-left corners int [FRAMES][n][sprites][2] and sizes [n][sprites] of moving squares."""
    rng = np.random.default_rng(seed)
    ns, vm = case["sprites"], case["vmax"]
    size = rng.integers(case["smin"], case["smax"] + 1, size=(n, ns))
    hi = np.stack([case["h"] - size, case["w"] - size], -1)
    pos = rng.integers(0, hi + 1)
    steps = [(dy, dx) for dy in range(-vm, vm + 1) for dx in range(-vm, vm + 1) if dy or dx]
    steps = np.asarray(steps)[rng.integers(0, len(steps), size=(FRAMES, n, ns))]
    out = [pos]
    for t in range(1, FRAMES):
        p = np.abs(out[-1] + steps[t])
        out.append(np.where(p > hi, 2 * hi - p, p))
    return np.stack(out), size


def _paint(frames, case, pos, size):
    """255-valued squares onto uint8 frames [FRAMES][n][1][h][w]."""
    dev = frames.device
    y = torch.arange(case["h"], device=dev).view(1, 1, -1, 1)
    x = torch.arange(case["w"], device=dev).view(1, 1, 1, -1)
    p, s = torch.from_numpy(pos).to(dev), torch.from_numpy(size).to(dev)
    for i in range(case["sprites"]):
        y0, x0, d = (v[..., None, None] for v in (p[:, :, i, 0], p[:, :, i, 1], s[:, i]))
        frames[:, :, 0].masked_fill_(((y >= y0) & (y < y0 + d)) & ((x >= x0) & (x < x0 + d)), 255)


def _dirty_share(case):
    """Share of pixels that change, layers 0..L, over a few streams' frames (1 where a pass is dense)."""
    layers = _layers(case)
    if case["kind"] in ("full", "update"):
        return [1.0] * (len(layers) + 1)
    if case["kind"] == "variants":
        d = torch.zeros(1, 1, case["h"], case["w"])
        y, x = (case["h"] - case["patch"]) // 2, (case["w"] - case["patch"]) // 2
        d[:, :, y:y + case["patch"], x:x + case["patch"]] = 1
    else:
        n = min(4, case["n"])
        f = torch.from_numpy(np.random.default_rng(1).integers(0, 256, (1, n, 1, case["h"], case["w"]), np.uint8))
        f = f.repeat(FRAMES, 1, 1, 1, 1)
        _paint(f, case, *_positions(case, n, 1))
        d = (f[1:] != f[:-1]).float().flatten(0, 1)
        if NETS[case["net"]][0] > 1:             # a stacked input changes where any of its frames does
            d = d.view(FRAMES - 1, n, 1, case["h"], case["w"]).amax(0)
    share = [float(d.mean())]
    for _ci, _co, k, s, p, _h, _w in layers:
        d = F.max_pool2d(F.pad(d, (p, p, p, p)), k, s)
        share.append(float(d.mean()))
    return share


def work(case):
    """Bytes and operations of one pass that the path cannot do without: frames and the cached input read, the
    changed outputs of each layer written and what they reach read, and the weights; the gradient is dense."""
    layers, share, n = _layers(case), _dirty_share(case), case["n"]
    act = 2 if case["act"] == "bf16" else 4
    px = case["h"] * case["w"]
    frame = px * (1 if case["frame"] == "u8" else 4)
    nbytes = frame + px * 4.0 * share[0] if case["kind"] == "variants" else n * (frame + px * 4.0)
    flops = 0.0
    before = (px, 1)
    for l, (ci, co, k, _s, _p, h, w) in enumerate(layers):
        macs, outs = n * h * w * co * ci * k * k, n * h * w * co
        flops += 2 * macs * share[l + 1]
        reads = n * before[0] * before[1] * min(1.0, share[l + 1]) * (4 if l == 0 else act)
        nbytes += outs * share[l + 1] * act + reads + co * ci * k * k * act
        if case["kind"] == "train":
            flops += 2 * macs * (1 if l == 0 else 2)
            nbytes += 4 * (outs + n * before[0] * before[1] + 2 * co * ci * k * k)
        before = (h * w, co)
    feats = before[0] * before[1]
    flops += 2 * n * feats * case["n_out"] * share[-1]
    nbytes += feats * case["n_out"] * act * min(1.0, n * share[-1]) + 4 * n * case["n_out"]
    if case["kind"] == "train":
        flops += 4 * n * feats * case["n_out"]
        nbytes += 8 * feats * case["n_out"]
    if case["kind"] == "update":
        nbytes += 12 * (feats * case["n_out"] + sum(co * ci * k * k for ci, co, k, *_ in layers))
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- inputs

def _inputs(case, seed):
    """Weights, frames [FRAMES][n or 1][1][h][w] and what else the kind needs, from the seed alone, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=0.05):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=g)

    layers, n = _layers(case), case["n"]
    conv_w = [normal(co, ci, k, k) for ci, co, k, *_ in layers]
    conv_b = [normal(co) for _ci, co, *_ in layers]
    _ci, cl, _k, _s, _p, hl, wl = layers[-1]
    dense_w, dense_b = normal(case["n_out"], cl * hl * wl, std=0.02), normal(case["n_out"])
    streams = 1 if case["kind"] == "variants" else n
    back = torch.randint(0, 256, (1, streams, 1, case["h"], case["w"]), generator=g, device="cuda", dtype=torch.uint8)
    frames = back.repeat(FRAMES, 1, 1, 1, 1)
    _paint(frames, case, *_positions(case, streams, seed))
    if case["frame"] == "f32":
        frames = frames.float() / 255.0
    got = {"weights": (conv_w, conv_b, dense_w, dense_b), "frames": frames}
    if case["kind"] == "train":
        got["actions"] = torch.randint(0, case["n_out"], (n,), generator=g, device="cuda", dtype=torch.int32)
        got["returns"] = torch.empty(n, device="cuda").uniform_(-1.0, 1.0, generator=g)
    if case["kind"] == "update":
        got["grads"] = torch.cat([normal(t.numel(), std=1.0)
                                  for w, b in [*zip(conv_w, conv_b), (dense_w, dense_b)] for t in (w, b)])
    if case["kind"] == "variants":
        p = case["patch"]
        side = math.ceil(math.sqrt(n))           # a grid of places over the whole frame
        y = torch.linspace(0, case["h"] - p, side).round().int().repeat_interleave(side)[:n]
        x = torch.linspace(0, case["w"] - p, side).round().int().repeat(side)[:n]
        got["boxes"] = torch.stack([y, x, y + p, x + p], 1).cuda()
        got["offsets"] = torch.arange(n + 1, dtype=torch.int32, device="cuda")
        got["patch"] = torch.zeros_like(frames[0])
        got["max_tiles"] = ((p + 2 * len(layers) + 2) // 4 + 1) ** 2      # 4x4 tiles a grown patch can touch
    return got


def prepare(case, seed):
    d = _inputs(case, seed)
    stack, convs = NETS[case["net"]]
    conv_w, conv_b, dense_w, dense_b = d.pop("weights")
    host = ([w.cpu().numpy() for w in conv_w], [b.cpu().numpy() for b in conv_b], dense_w.cpu().numpy(),
            dense_b.cpu().numpy())
    streams = 1 if case["kind"] == "variants" else case["n"]
    net = ReuseNet(1, case["h"], case["w"], convs, case["n_out"], streams, host, act_dtype=case["act"], stack=stack,
                   head=case["head"], fuse_first=case["kind"] != "train")
    if case["kind"] not in ("full", "update"):
        net.full(d["frames"][0])
    if case["kind"] == "train":
        d["grads"] = net.new_grads()
    return dict(d, case=case, net=net, passes=0)


def run(state):
    net, kind = state["net"], state["case"]["kind"]
    if kind == "variants":
        return net.variants(0, state["boxes"], state["offsets"], state["patch"], max_tiles=state["max_tiles"])
    state["passes"] += 1
    t = state["passes"] % (2 * FRAMES - 2)
    x = state["frames"][min(t, 2 * FRAMES - 2 - t)]
    if kind == "step":
        return net.step(x)
    if kind == "full":
        return net.full(x)
    if kind == "update":
        # The sign alternates, so that the weights stay where a program's are.
        net.sgd_step(state["grads"], LR if state["passes"] % 2 else -LR)
        return net.step(x)
    logits = net.step(x)
    dlogits = net.reinforce_dlogits(logits, state["actions"], state["returns"])
    return {"logits": logits, "dlogits": dlogits, "grads": net.backward(dlogits, state["grads"])}


# ---------------------------------------------------------------- float64

def _forward64(case, weights, x):
    """Logits of inputs x [n][cin][h][w] in float64, and each layer's (input, pre-activation)."""
    conv_w, conv_b, dense_w, dense_b = weights
    kept = []
    for (ci, co, k, s, p, h, w), cw, cb in zip(_layers(case), conv_w, conv_b):
        z = torch.stack([(cw.view(co, -1) @ F.unfold(v[None], k, padding=p, stride=s)[0]).view(co, h, w) for v in x])
        z += cb.view(1, -1, 1, 1)
        kept.append((x, z))
        x = z.clamp_min(0.0)
    return x.flatten(1) @ dense_w.t() + dense_b, kept


def _backward64(case, weights, kept, dlogits, grads):
    """Adds the gradient of sum(dlogits * logits) to grads (the weights in order, each (weight, bias))."""
    conv_w, _conv_b, dense_w, _dense_b = weights
    feats = kept[-1][1].clamp_min(0.0)
    grads[-1][0].add_(dlogits.t() @ feats.flatten(1))
    grads[-1][1].add_(dlogits.sum(0))
    dz = (dlogits @ dense_w).view_as(feats) * (kept[-1][1] > 0)
    for l in range(len(kept) - 1, -1, -1):
        x = kept[l][0]
        co, ci = conv_w[l].shape[:2]
        for v, d in zip(x, dz):                  # per frame: the unfolded input is nine times the input
            grads[l][0].add_((d.flatten(1) @ F.unfold(v[None], 3, padding=1)[0].t()).view(co, ci, 3, 3))
        grads[l][1].add_(dz.sum((0, 2, 3)))
        if l:
            back = conv_w[l].flip(2, 3).transpose(0, 1).reshape(ci, -1)
            dx = torch.stack([(back @ F.unfold(d[None], 3, padding=1)[0]).view(ci, *d.shape[1:]) for d in dz])
            dz = dx * (kept[l - 1][1] > 0)


def exact(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    stack, _convs = NETS[case["net"]]
    bf16 = case["act"] == "bf16"

    def wide(t, quantise=True):
        return (t.bfloat16() if bf16 and quantise else t).double()

    conv_w, conv_b, dense_w, dense_b = d["weights"]
    weights = ([wide(w) for w in conv_w], [wide(b, False) for b in conv_b], wide(dense_w), wide(dense_b, False))
    if kind == "update":
        flat = [t for w, b in [*zip(*weights[:2]), weights[2:]] for t in (w, b)]
        for t, g in zip(flat, d["grads"].split([t.numel() for t in flat])):
            t.sub_(LR * g.double().view_as(t))

    def values(x):
        return wide(x.float() / 255.0 if x.dtype == torch.uint8 else x)

    first = values(d["frames"][0])
    if kind == "variants":
        def inputs(i, j):
            x = first.repeat(j - i, 1, 1, 1)
            for v, (y0, x0, y1, x1) in zip(x, d["boxes"][i:j].tolist()):
                v[:, y0:y1, x0:x1] = 0.0
            return x
    else:
        second = values(d["frames"][1])
        old = second if kind in ("full", "update") else first      # an unprimed slot takes its frame as all four

        def inputs(i, j):
            return torch.cat([old[i:j]] * (stack - 1) + [second[i:j]], 1)

    logits, dlogits = [], []
    grads = [(torch.zeros_like(w), torch.zeros_like(b)) for w, b in [*zip(*weights[:2]), weights[2:]]]
    for i in range(0, case["n"], 8):
        j = min(i + 8, case["n"])
        z, kept = _forward64(case, weights, inputs(i, j))
        logits.append(z)
        if kind == "train":
            hot = F.one_hot(d["actions"][i:j].long(), case["n_out"])
            dlogits.append(d["returns"][i:j, None].double() * (torch.softmax(z, 1) - hot))
            _backward64(case, weights, kept, dlogits[-1], grads)
    logits = torch.cat(logits)
    if kind != "train":
        return logits
    return {"logits": logits, "dlogits": torch.cat(dlogits),
            "grads": torch.cat([t.flatten() for pair in grads for t in pair])}


def tolerance(case):
    # About four times what the path is off from float64 (float32: up to 7e-7; bfloat16, where every cached activation
    # is rounded: 3e-3).  Gradients, up to 3e-4: a pre-activation within rounding of 0 may take either derivative of the
    # rectifier, which changes that element's whole gradient.
    if case["act"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": 1.5e-3, "max": 3e-2} if case["kind"] == "train" else {"rel": 4e-6}
