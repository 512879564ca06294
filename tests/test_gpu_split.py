"""Float32 layers on the bf16 matrix cores with split operands: group sizes and
their remainders against the oracle and each other, and values the split cannot
carry (infinities, magnitudes that round up to infinity in bf16)."""
import numpy as np
import pytest

import oracle
from synth import frames as synth
from gpu_util import ATOL_F32, make_net, oracle_net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


# 88 tiles a stream (ragged bottom row): groups of 4 (88 and 440 tiles), of 8
# (1144) and of 16 (2112), whose last groups are part empty on every XCD's share.
@pytest.mark.parametrize("n", [1, 5, 13, 24])
def test_group_sizes(torch, n):
    wl = synth.Workload(cid=201, streams=n, frames=1, h=42, w=32, convs=(64, 128, 128), n_out=18,
                        n_sprites=3, smin=3, smax=6, vmin=1, vmax=3)
    weights = synth.net_weights(wl, bias_std=0.05)
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(n), frames=1))[0][:, None]
    dev = torch.from_numpy(x).cuda()
    a, b, one = make_net(wl, n, weights), make_net(wl, n, weights), make_net(wl, 1, weights)
    full = a.full(dev).cpu().numpy()
    step = b.step(dev).cpu().numpy()                     # all dirty: the same tiles by list
    assert np.array_equal(full.view(np.uint32), step.view(np.uint32))
    for i in sorted({0, n // 2, n - 1}):
        alone = one.full(dev[i:i + 1].contiguous()).cpu().numpy()
        assert np.array_equal(full[i:i + 1].view(np.uint32), alone.view(np.uint32)), i
        ref, acts = oracle.forward(oracle_net(wl), *weights, x[i:i + 1], want_acts=True)
        assert np.abs(full[i] - ref[0]).max() <= ATOL_F32
        for l in (2, 3):
            assert np.array_equal(a.activation(i, l), one.activation(0, l)), (i, l)
            assert np.abs(a.activation(i, l) - acts[l - 1][0]).max() <= ATOL_F32, (i, l)
    for net in (a, b, one):
        net.close()


def _weights(wl, rng, scale):
    """Layer 1 copies the frame into channel 0 (others: -frame and plain random taps); later layers random."""
    w = list(synth.net_weights(wl, bias_std=0.05))
    cw = [np.array(v) for v in w[0]]
    cw[0][0] = cw[0][1] = 0.0
    cw[0][0, 0, 1, 1], cw[0][1, 0, 1, 1] = 1.0, -1.0
    for l in range(1, len(cw)):
        cw[l] = (rng.normal(0.0, scale, cw[l].shape)).astype(np.float32)
    return (cw, *w[1:])


def _check_layers(torch, wl, weights, x, fuse=True):
    """Every layer of a dense pass of two frames against torch's float32 convolution of the layer's own input."""
    from paper_1909_05632_amd import ReuseNet
    import torch.nn.functional as F
    net = ReuseNet(1, wl.h, wl.w, wl.convs, wl.n_out, 2, weights, fuse_first=fuse)
    net.full(torch.from_numpy(x).cuda())
    cur = torch.from_numpy(x)
    for l in range(1, len(wl.convs) + 1):
        w, b = torch.from_numpy(weights[0][l - 1]), torch.from_numpy(weights[1][l - 1])
        pad = F.pad(cur, (1, 1, 1, 1))                    # zeros that are multiplied, as the kernels do
        z = F.conv2d(pad, w, b)
        size = F.conv2d(pad.abs(), w.abs(), b.abs()).numpy()   # sum of the terms' magnitudes
        want = torch.clamp_min(z, 0.0).numpy()
        got = np.stack([net.activation(i, l) for i in range(2)])
        known = ~np.isnan(z.numpy())
        fin = known & np.isfinite(want) & np.isfinite(size)
        assert np.array_equal(np.isinf(got[known]), np.isinf(want[known])), l
        assert np.all((got[~known] == 0.0) | ~np.isfinite(got[~known])), l
        with np.errstate(over="ignore"):
            assert np.all(np.abs(got[fin] - want[fin]) <= 1152 * 2.0 ** -24 * size[fin] + 1e-30), l
        cur = torch.from_numpy(got)                       # the next layer's input as the GPU has it
    net.close()


@pytest.mark.parametrize("convs", [(64, 128, 128), (40, 80)])
@pytest.mark.parametrize("value", [3.4e38, -3.4e38, np.inf, -np.inf])
def test_values_beyond_the_split(torch, value, convs):
    # One pixel of the frame holds `value`.  Plain float32 arithmetic (torch on
    # the CPU, sums in another order) gives the expected result wherever it is
    # not NaN; where it is, the GPU's ReLU may give NaN or 0 (the sign of a NaN).
    # 3.4e38 is finite in float32 and infinite in bf16; the layer weights keep
    # its products and their sums finite.  Tolerance: 1152 float32 roundings.
    wl = synth.Workload(cid=202, streams=2, frames=1, h=20, w=24, convs=convs, n_out=18)
    weights = _weights(wl, np.random.default_rng(5), 1e-4)
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(2), frames=1))[0][:, None]
    x[0, 0, 9, 10] = value
    _check_layers(torch, wl, weights, x)


# A weight, or a bias, of each later layer that no bf16 holds: 3.4e38 is finite
# in float32 (the frame's values keep its products finite).
@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("convs", [(64, 128, 128), (40, 80)])
@pytest.mark.parametrize("value", [3.4e38, -3.4e38, np.inf, -np.inf, np.nan])
def test_weights_beyond_the_split(torch, value, convs, fuse):
    wl = synth.Workload(cid=211, streams=2, frames=1, h=20, w=24, convs=convs, n_out=18)
    weights = _weights(wl, np.random.default_rng(12), 1e-4)
    for l in range(1, len(convs)):
        weights[0][l][5, 3, 1, 1] = weights[0][l][70, 9, 0, 2] = value
        weights[1][l][11] = value
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(2), frames=1))[0][:, None] * np.float32(0.01)
    _check_layers(torch, wl, weights, x, fuse)


# Head partials by position: groups of 1 item (88 tiles), 5 (2112) and 18 (8800)
# a block, one to three column blocks; a stream's logits are those it has alone,
# and the oracle's.
@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("n_out", [6, 18, 40])
def test_head_groups(torch, act, n_out):
    wl = synth.Workload(cid=203, streams=100, frames=1, h=42, w=32, convs=(64, 128, 128), n_out=n_out,
                        n_sprites=3, smin=3, smax=6, vmin=1, vmax=3)
    weights = synth.net_weights(wl, bias_std=0.05)
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(100), frames=1))[0][:, None]
    dev = torch.from_numpy(x).cuda()
    net, one = make_net(wl, 100, weights, act_dtype=act), make_net(wl, 1, weights, act_dtype=act)
    got = {n: net.full(dev[:n].contiguous()).cpu().numpy() for n in (24, 100)}
    for i in (0, 11, 23):
        alone = one.full(dev[i:i + 1].contiguous()).cpu().numpy()[0]
        assert np.array_equal(alone, got[24][i]) and np.array_equal(alone, got[100][i]), i
        ref, _ = oracle.forward(oracle_net(wl, act == "bf16"), *weights, x[i:i + 1])
        tol = ATOL_F32 if act == "f32" else 1e-2 * np.abs(ref).max()
        assert np.abs(alone - ref[0]).max() <= tol, i
    net.close()
    one.close()


def _chain(x, w, b):
    """Pre-activations of a 40 -> 80 layer for x [40][H][W], summed one float32 fma at a time in the float32
    kernel's order (position, 16-channel block, k-step, quarter): float64 holds a product exactly, and its
    sum with a float32 before rounding to within 2^-53 of itself."""
    H, W = x.shape[1:]
    xp = np.zeros((40, H + 2, W + 2))
    xp[:, 1:-1, 1:-1] = x
    acc = np.zeros((80, H, W), np.float32)
    for kpos in range(9):
        for blk, steps in ((0, 4), (1, 4), (2, 2)):
            for j in range(steps):
                for kq in range(4):
                    c = 16 * blk + steps * kq + j
                    win = xp[c, kpos // 3:kpos // 3 + H, kpos % 3:kpos % 3 + W]
                    acc = (w[:, c, kpos // 3, kpos % 3].astype(np.float64)[:, None, None] * win + acc).astype(np.float32)
    return acc + b[:, None, None]


def _uneven(weights, big=2.0 ** 20, small=2.0 ** -20):
    """The same weights with a loud, a quiet and a silent channel in the last conv layer."""
    cw, cb = [np.array(v) for v in weights[0]], [np.array(v) for v in weights[1]]
    for c, f in ((3, big), (7, small), (11, 0.0)):
        cw[-1][c] *= np.float32(f)
        cb[-1][c] *= np.float32(f)
    return (cw, cb, *weights[2:])


def _column_size(x, w):
    """Largest magnitude of a channel's first and last partial sums over the 4 pixels of a tile column: K in octets
    of channels, octet g at kernel position g / 5, twelve octets (the last one nine) a partial sum."""
    H, W = x.shape[1:]
    xp = np.zeros((40, -(-H // 4) * 4 + 2, W + 2))
    xp[:, 1:H + 1, 1:-1] = x
    part = np.zeros((2, 80, xp.shape[1] - 2, W))
    for g in (*range(12), *range(36, 45)):
        pos, c = g // 5, 8 * (g % 5)
        win = xp[c:c + 8, pos // 3:pos // 3 + part.shape[2], pos % 3:pos % 3 + W]
        part[g // 36] += np.tensordot(w[:, c:c + 8, pos // 3, pos % 3].astype(np.float64), win, 1)
    size = np.abs(part).max(0).reshape(80, -1, 4, W).max(2)
    return np.repeat(size, 4, 1)[:, :H]


@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("uneven", [False, True])
def test_decisions_near_zero_are_float32s(torch, fuse, uneven):
    # Results within 2^-19 of 0 relative to the largest of their channel's first
    # and last partial sums in their tile column come from the float32 sum: up
    # to half of that they are the chain's, bit for bit, whatever the sizes of
    # the other channels are; the others only to rounding.
    from paper_1909_05632_amd import ReuseNet
    wl = synth.Workload(cid=205, streams=12, frames=1, h=101, w=80, convs=(40, 80), n_out=6)
    weights = synth.net_weights(wl, bias_std=0.05)
    if uneven:
        weights = _uneven(weights)
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(12), frames=1))[0][:, None]
    net = ReuseNet(1, wl.h, wl.w, wl.convs, 6, 12, weights, fuse_first=fuse)
    net.full(torch.from_numpy(x).cuda())
    seen = 0
    for i in range(12):
        a1 = net.activation(i, 1)
        z, size = _chain(a1, weights[0][1], weights[1][1]), _column_size(a1, weights[0][1])
        near = np.abs(z) < size * 2.0 ** -20
        tile = np.pad(np.abs(z) < size * 2.0 ** -18, ((0, 0), (0, 3), (0, 0))).reshape(80, 26, 4, 20, 4).sum((0, 2, 4))
        assert tile.max() <= 4                            # each taken one by one
        got, want = net.activation(i, 2), np.maximum(z, np.float32(0))
        assert np.array_equal(got[near], want[near])
        bound = 360 * 2.0 ** -24 * np.abs(weights[0][1]).sum((1, 2, 3)) * np.abs(a1).max()
        assert np.all(np.abs(got - want) <= bound[:, None, None])
        seen += int(near.sum())
    assert seen > 0
    net.close()


@pytest.mark.parametrize("fuse", [True, False])
def test_time_of_a_layer_whatever_its_values(torch, fuse):
    # Channels of very different size: a rule that takes float32 sums by the
    # size of other channels made this 10 times slower; the bound is far from
    # both.  Medians of dense passes, weights in turn.
    from paper_1909_05632_amd import ReuseNet
    n = 64
    wl = synth.Workload(cid=208, streams=n, frames=1, h=105, w=80, convs=(40, 80), n_out=6)
    even = synth.net_weights(wl, bias_std=0.05)
    x = torch.from_numpy(synth.to_f32(synth.sprite_batch(wl, streams=range(n), frames=1))[0][:, None]).cuda()
    nets = [ReuseNet(1, wl.h, wl.w, wl.convs, 6, n, w, fuse_first=fuse) for w in (even, _uneven(even))]
    ms = [[], []]
    for _ in range(12):
        for net, t in zip(nets, ms):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            net.full(x)
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
    assert np.median(ms[1]) < 1.5 * np.median(ms[0]), ms
    for net in nets:
        net.close()


# Options of a net: its convs, whether layer 1 is folded into layer 2.
ONE_ARITHMETIC = [((40, 80), True), ((40, 80), False), ((64, 128, 128), True), ((64, 128, 128), False)]


@pytest.mark.parametrize("n_out", [6, 18])
@pytest.mark.parametrize("convs,fuse", ONE_ARITHMETIC)
def test_step_full_and_variants_agree(torch, convs, fuse, n_out):
    # Of one net a step, a dense pass and a variant of the same frame give the
    # same bits, and a variant that rewrites the base's own pixels gives the
    # base's; in a 40->80 layer but for results next to 0, which variants do not
    # take from the float32 sum: a few results a frame, each off by 2^-19 of its
    # partial sums at most, times a dense weight.  16 ragged frames, variant i =
    # slot 0 with frame i in its boxes.
    from paper_1909_05632_amd import ReuseNet
    wl = synth.Workload(cid=209, streams=16, frames=1, h=101, w=80, convs=convs, n_out=n_out,
                        n_sprites=3, smin=3, smax=6, vmin=1, vmax=3)
    weights = synth.net_weights(wl, bias_std=0.05)
    x = torch.from_numpy(synth.to_f32(synth.sprite_batch(wl, streams=range(16), frames=1))[0][:, None]).cuda()
    net = ReuseNet(1, wl.h, wl.w, convs, n_out, 16, weights, fuse_first=fuse)
    other = ReuseNet(1, wl.h, wl.w, convs, n_out, 16, weights, fuse_first=fuse)
    full, step = net.full(x), other.step(x)
    assert torch.equal(full, step)
    whole = torch.tensor([[0, 0, wl.h, wl.w]] * 16, dtype=torch.int32, device="cuda")
    part = torch.tensor([[3 * i, 2 * i, 3 * i + 9, 2 * i + 14] for i in range(16)], dtype=torch.int32, device="cuda")
    off = torch.arange(17, dtype=torch.int32, device="cuda")
    tiles = 26 * 20

    def same(got, want):
        return torch.equal(got, want) if convs[0] == 64 else float((got - want).abs().max()) <= 1e-6 * float(want.abs().max())

    assert same(net.variants(0, whole, off, x, max_tiles=tiles), full)
    # 64 variants: 33280 tiles a layer, the staged kernel's groups of 8
    many = net.variants(0, whole.repeat(4, 1), torch.arange(65, dtype=torch.int32, device="cuda"), x.repeat(4, 1, 1, 1),
                        max_tiles=tiles)
    assert same(many, full.repeat(4, 1))
    assert same(net.variants(0, part, off, x[:1], max_tiles=tiles), full[:1].expand(16, n_out))
    net.close()
    other.close()


@pytest.mark.parametrize("convs,h,w", [((40, 80), 42, 32), ((64, 128, 128), 42, 32), ((40, 80), 13, 20)])
def test_gradients_add_over_batches(torch, convs, h, w):
    # Input gradients in groups of 16, 8 and 4 tiles (24, 13 and 1 streams of 88
    # tiles) and weight gradients over teams of even and odd tile counts: the
    # gradient of a batch is the sum of its parts' (each checked against the
    # oracle in test_gpu_train.py).  Tolerance: float32 sums in another order,
    # relative to each tensor's largest.
    from paper_1909_05632_amd import ReuseNet
    n = 37
    wl = synth.Workload(cid=206, streams=n, frames=1, h=h, w=w, convs=convs, n_out=18)
    weights = synth.net_weights(wl, bias_std=0.05)
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(n), frames=1))[0][:, None]
    g = torch.from_numpy(np.random.default_rng(6).normal(size=(n, 18)).astype(np.float32)).cuda()
    net = ReuseNet(1, h, w, convs, 18, n, weights, fuse_first=False)
    net.full(torch.from_numpy(x).cuda())
    whole = net.backward(g, net.new_grads()).clone()
    parts = net.new_grads()
    for a, b in ((0, 13), (13, 36), (36, 37)):
        ids = torch.arange(a, b, dtype=torch.int32, device="cuda")
        net.backward(g[a:b].contiguous(), parts, stream_ids=ids, accumulate=True)
    for u, v in zip(net.split_grads(whole), net.split_grads(parts)):
        for p, q in zip(u, v) if isinstance(u, list) else [(u, v)]:
            assert float((p - q).abs().max()) <= 2e-6 * float(p.abs().max()) + 1e-12
    net.close()


@pytest.mark.parametrize("convs", [(40, 80), (64, 128, 128)])
@pytest.mark.parametrize("n,h,w", [(2, 14, 16), (5, 45, 40)])
def test_gradients_of_infinities(torch, n, h, w, convs):
    # An infinite logit gradient: products and sums of every layer's gradients
    # are infinite or NaN exactly where IEEE arithmetic makes them so (float64
    # gives the same classes), not where operands split in three cancel.  4
    # teams of tiles, two of them without an infinity, and 75 (more than a
    # wave's lanes); weight gradients of one block and of several a team, input
    # gradients to 40, 64 and 128 channels.
    wl = synth.Workload(cid=207, streams=n, frames=1, h=h, w=w, convs=convs, n_out=6)
    weights = synth.net_weights(wl, bias_std=0.05)
    x = synth.to_f32(synth.sprite_batch(wl, streams=range(n), frames=1))[0][:, None]
    net = make_net(wl, n, weights)
    net.full(torch.from_numpy(x).cuda())
    g = np.random.default_rng(8).normal(size=(n, 6)).astype(np.float32)
    g[n - 1, 1] = np.inf
    cw, cb, _dw, _db = net.split_grads(net.backward(torch.from_numpy(g).cuda(), net.new_grads()))
    acts = [x] + [np.stack([net.activation(i, l) for i in range(n)]) for l in range(1, len(convs) + 1)]

    def shifted(v):                                       # [3][3] views of v shifted by the kernel positions
        p = np.pad(v, ((0, 0), (0, 0), (1, 1), (1, 1)))
        return [[p[:, :, ky:ky + h, kx:kx + w] for kx in range(3)] for ky in range(3)]

    with np.errstate(invalid="ignore"):
        da = (g.astype(np.float64) @ weights[2]).reshape(acts[-1].shape)
        for l in range(len(convs), 0, -1):
            dz = np.where(acts[l] > 0, da, 0.0)
            prev = shifted(acts[l - 1].astype(np.float64))
            # (summed channel by channel: matrix products of infinities are left to numpy's plain loops)
            want = np.stack([np.stack([np.stack([(dz * v[:, None, c]).sum((0, 2, 3)) for c in range(v.shape[1])], 1)
                                       for v in row], -1) for row in prev], -2)
            for u, v in ((cw[l - 1].cpu().numpy(), want), (cb[l - 1].cpu().numpy(), dz.sum((0, 2, 3)))):
                assert np.array_equal(np.isnan(u), np.isnan(v)), l
                assert np.array_equal(np.isposinf(u), np.isposinf(v)) and np.array_equal(np.isneginf(u), np.isneginf(v)), l
            if l > 1:
                wt, back = weights[0][l - 1].astype(np.float64), shifted(dz)
                da = np.zeros(acts[l - 1].shape)
                for ky in range(3):
                    for kx in range(3):
                        for c in range(wt.shape[0]):
                            da += wt[None, c, :, 2 - ky, 2 - kx, None, None] * back[ky][kx][:, c, None]
    net.close()


def _phase_ms(torch, net, phase, call, runs=5):
    """Median time of a phase of a call, from the library's own events."""
    ms = []
    for _ in range(runs):
        net.set_profiling(True)
        call()
        torch.cuda.synchronize()
        ms.append(net.profile()[phase]["ms"])
        net.set_profiling(False)
    return float(np.median(ms))


# Slowest weight gradient of a batch with infinite or NaN logit gradients,
# relative to a finite one: 14.5 and 15 with the sums of 64 weights taken again
# by one wave in turn; 6.8 and less where a channel that is on in few tiles has
# infinite sums that never become NaN, 2.3 and 4.1 otherwise.
@pytest.mark.parametrize("convs,n,h,w", [((40, 80), 64, 105, 80), ((64, 128, 128), 16, 106, 92)])
def test_time_of_non_finite_weight_gradients(torch, convs, n, h, w):
    from paper_1909_05632_amd import ReuseNet
    wl = synth.Workload(cid=210, streams=n, frames=1, h=h, w=w, convs=convs, n_out=6)
    net = ReuseNet(1, h, w, convs, 6, n, synth.net_weights(wl, bias_std=0.05), fuse_first=False)
    net.full(torch.from_numpy(synth.to_f32(synth.sprite_batch(wl, streams=range(n), frames=1))[0][:, None]).cuda())
    g = torch.from_numpy(np.random.default_rng(9).normal(size=(n, 6)).astype(np.float32)).cuda()
    grads, one = net.new_grads(), g.clone()
    one[:, 0] = np.inf
    finite, *others = (_phase_ms(torch, net, "bwd_dw", lambda: net.backward(v, grads))
                       for v in (g, one, torch.full_like(g, np.inf), torch.full_like(g, np.nan)))
    assert max(others) < 10 * finite, (finite, others)
    net.close()


# Layers and calls with infinities or NaN in weights or logit gradients, times
# relative to the finite ones: up to 2 (input gradients) and 10 (forward) with
# every such result summed again one by one; 1, and up to 3.7 (40->80, infinities:
# a second pass over a tile's leading terms).
@pytest.mark.parametrize("convs,n,h,w", [((40, 80), 64, 105, 80), ((64, 128, 128), 16, 106, 92)])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_time_of_non_finite_split_layers(torch, value, convs, n, h, w):
    from paper_1909_05632_amd import ReuseNet
    wl = synth.Workload(cid=212, streams=n, frames=1, h=h, w=w, convs=convs, n_out=6)
    weights = synth.net_weights(wl, bias_std=0.05)
    x = torch.from_numpy(synth.to_f32(synth.sprite_batch(wl, streams=range(n), frames=1))[0][:, None]).cuda()
    g = torch.from_numpy(np.random.default_rng(9).normal(size=(n, 6)).astype(np.float32)).cuda()
    odd = ([np.array(v) for v in weights[0]], *weights[1:])
    odd[0][1][:, 0, 0, 0] = value
    ms = {}
    for name, wts in (("finite", weights), ("odd", odd)):
        net = ReuseNet(1, h, w, wl.convs, 6, n, wts)
        grads = net.new_grads()
        ms[name, "forward"] = _phase_ms(torch, net, "convN", lambda: net.full(x))
        ms[name, "weights"] = _phase_ms(torch, net, "bwd_dx", lambda: net.backward(g, grads))
        if name == "finite":
            ms[name, "gradients"] = ms[name, "weights"]
            ms["odd", "gradients"] = _phase_ms(torch, net, "bwd_dx", lambda: net.backward(torch.full_like(g, value), grads))
        net.close()
    for what in ("forward", "weights", "gradients"):
        assert ms["odd", what] < 5 * ms["finite", what], ms
