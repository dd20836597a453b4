"""fp32 convolutions and weight gradients in two fp16 parts per number (csrc/ranges.hpp, csrc/kernels_conv_parts.hpp, csrc/kernels_wgrad_parts.hpp):
every length of the runs in which leading products are summed, and numbers that two parts do not suit, against 64-bit sums.  bf16 convolutions of eight tiles
per wave against those of fewer."""
import os
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1302_1690_amd import mpcnn, workloads as wl
from test_gpu_conv_parts import activations, close_layers, reached

pytestmark = pytest.mark.gpu
C, MP, FC = wl.C, wl.MP, wl.FC

# filters and channels of the layer behind the first: sums of 512 products and a few more in both directions; three parts (1 x 1: blocks of fewer than four
# steps), runs of two chunks, a chunk, filter rows of a chunk (two, three, one) and, from 8 rows on, filter rows in blocks of fewer rows
SHAPES = [(1, 516, 520), (2, 128, 132), (3, 60, 64), (4, 32, 36), (5, 24, 40), (6, 16, 20), (7, 12, 16), (8, 8, 12), (11, 8, 8), (26, 8, 8)]


def gradient64(layers, patch, params, image, labels, pixw=None, logistic=False):
    """The flat gradient in 64 bits, pool-free nets with cross-entropy, and each layer's biases' places and root of the sum of squared deltas."""
    tensors, at, side, ci, fc, pre, places = [], 0, patch, 1, False, [], []
    x = torch.from_numpy(image).double()
    for i, (kind, m, k) in enumerate(layers):
        k = k if kind == C else (1 if fc else side)
        n = m * ci * k * k
        w = torch.from_numpy(params[at:at + n].astype(np.float64).reshape(m, ci, k, k)).requires_grad_()
        b = torch.from_numpy(params[at + n:at + n + m].astype(np.float64)).requires_grad_()
        tensors += [w, b]
        x = torch.nn.functional.conv2d(x, w, b)
        x.retain_grad()
        pre.append(x)
        places.append(slice(at + n, at + n + m))
        if i < len(layers) - 1:
            x = torch.sigmoid(x) if logistic else torch.tanh(x)
        at += n + m
        side, ci, fc = (side - k + 1 if kind == C else 1), m, fc or kind == FC
    c = (patch - 1) // 2
    window = lambda t: torch.from_numpy(t)[:, c:c + x.shape[2], c:c + x.shape[3]]
    loss = torch.nn.functional.cross_entropy(x, window(labels).long(), reduction="none")
    (loss if pixw is None else loss * window(pixw).double()).sum().backward()
    return torch.cat([t.grad.reshape(-1) for t in tensors]).numpy(), [(p, float(z.grad.square().sum().sqrt())) for p, z in zip(places, pre)]


def far_maps(got, want, layers, patch, maps):
    """Largest relative distance (2-norm) of the gradient of one map by itself: (layer, "out" or "in", map)."""
    side, ci, at, worst, fc = patch, 1, 0, 0.0, False
    for layer, (kind, m, k) in enumerate(layers):
        k = k if kind == C else (1 if fc else side)
        n = m * ci * k * k
        g, w = (v[at:at + n].reshape(m, ci, k * k) for v in (got, want))
        for at_layer, way, i in maps:
            if at_layer == layer:
                a, b = (g[i], w[i]) if way == "out" else (g[:, i], w[:, i])
                worst = max(worst, np.linalg.norm(a - b) / np.linalg.norm(b))
        at, ci, fc, side = at + n + m, m, fc or kind == FC, side - k + 1
    return worst


def case(k, c0, c1, size, seed=3, hidden=24):
    layers = ((C, c0, 3), (C, c1, k), (FC, hidden, 0), (FC, 2, 0))
    patch = k + 4
    rng = np.random.default_rng(seed)
    H, W = patch + size, patch + size + 5
    image = rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)
    labels = rng.integers(0, 2, (1, H, W)).astype(np.int32)
    params, ci = [], 1
    for m, f in ((c0, 3), (c1, k), (hidden, 3), (2, 1)):
        params.append(rng.uniform(-1, 1, m * ci * f * f + m) * 1.5 / np.sqrt(ci * f * f))
        ci = m
    return layers, patch, np.concatenate(params).astype(np.float32), image, labels


def gradient(layers, patch, params, image, labels, pixw=None, logistic=False):
    net = mpcnn.Net(layers, 1, patch)
    net.set_params(params)
    net.set_activation("logistic" if logistic else "tanh")
    net.seg_backward(torch.from_numpy(image).cuda(), torch.from_numpy(labels).cuda(), pixw=None if pixw is None else torch.from_numpy(pixw).cuda())
    got = net.get_grads().astype(np.float64)
    plan = net.plan_describe(1, image.shape[2], image.shape[3], True)
    net.close()
    return got, plan


def bound(layers, patch):
    """A gradient's terms are products of activations and deltas, each of which has passed up to three sums of up to K products: a sum's error is at most
    as large as that of fp32 additions, sqrt(K / 3) 2^-24 of its terms' root of squares, and the squashing function's 1.2e-7 of 1, which a slope
    (1 - y^2 where y is near 1) carries over whole.  Five of the larger ones together."""
    side, ci, most, fc = patch, 1, 0, False
    for kind, m, k in layers:
        k = k if kind == C else (1 if fc else side)
        most = max(most, k * k * max(ci, m))
        ci, fc, side = m, fc or kind == FC, side - k + 1
    return 5 * max(np.sqrt(most / 3) * 2.0 ** -24, 1.2e-7)


@pytest.mark.parametrize("k,c0,c1", SHAPES)
def test_runs_of_every_length(k, c0, c1):
    args = case(k, c0, c1, 34)
    got, plan = gradient(*args)
    convs = [line for line in plan.splitlines() if "forward: " in line or "data gradient: " in line]
    assert sum("or two of fp16" in line for line in convs) >= (2 if k > 1 else 0), plan
    want = gradient64(*args)[0]
    assert close_layers(got, want, args[0], args[1]) <= bound(args[0], args[1])


# how the numbers of a layer are spread, and whose gradients show it
SPREADS = {"tiny_input_map": (2.0 ** -24, [(0, "out", 3), (1, "in", 3)]), "tinier_input_map": (2.0 ** -60, [(0, "out", 3), (1, "in", 3)]), "tiny_output_map": (2.0 ** -24, [(1, "out", 7), (2, "in", 7)]),
           "one_large_weight": (2.0 ** 20, []), "a_large_map": (2.0 ** 30, []), "class_weight": (2.0 ** -30, [(2, "out", 9)]),
           "class_weight_and_its_own_maps": (2.0 ** -30, [(2, "out", 9)] + [(1, "out", i) for i in range(4)]),
           "tiny_class_weight_and_its_own_maps": (2.0 ** -60, [(2, "out", 9)] + [(1, "out", i) for i in range(4)])}


@pytest.mark.parametrize("what", list(SPREADS))
@pytest.mark.parametrize("logistic", [False, True])
def test_numbers_that_do_not_suit_two_parts(what, logistic):
    """Input maps whose weights are 2^-24 and 2^-60 of the others, an output map of which the layer above sees 2^-24, one weight of 2^20, a map 2^30 times the others, a hidden unit whose
    class weights are 2^-30 or 2^-60 of the others, and one on which maps of the layer below depend alone.  Layers as a whole (bound), and the maps concerned by themselves: labels are random, so that a map's
    gradient over N positions is what is left of N terms, of the order of their root, and errors that all positions share (2e-7 of a term, at most 4e-7) may be sqrt(N) as large."""
    hidden = 128
    layers, patch, params, image, labels = case(3, 60, 64, 70 if "large" in what else 200, hidden=hidden)
    first, (size, maps) = 60 * 9 + 60, SPREADS[what]
    second = params[first:first + 64 * 60 * 9].reshape(64, 60, 9)      # (views)
    third = params[first + 64 * 60 * 9 + 64:][:hidden * 64 * 9].reshape(hidden, 64, 9)
    classes = params[-2 * hidden - 2:-2].reshape(2, hidden)
    if what.endswith("input_map"):
        second[:, 3] *= size
    elif what == "tiny_output_map":
        third[:, 7] *= size
    elif what == "one_large_weight":
        second[10, 20, 4] = size
    elif what == "a_large_map":
        second[5] *= size
    else:
        classes[:, 9] *= size
        if what.endswith("own_maps"):                                  # (maps 0 to 3 lead to unit 9 only)
            third[:9, :4] = 0
            third[10:, :4] = 0
    got, plan = gradient(layers, patch, params, image, labels, logistic=logistic)
    lines = [line for line in plan.splitlines() if "or two of fp16" in line]
    assert [sum(way in line for line in lines) for way in ("forward", "data gradient", "weight gradient")] == [2, 2, 0 if "large" in what else 1], plan
    want = gradient64(layers, patch, params, image, labels, logistic=logistic)[0]
    # (the map of one large weight is saturated but where its sum, off by 2^20 2^-24, is near 0: seen in the layer below, in any arithmetic)
    assert close_layers(got, want, layers, patch) <= (8 if what == "one_large_weight" else 1) * bound(layers, patch)
    if maps:
        assert far_maps(got, want, layers, patch, maps) <= np.sqrt(labels.size) * 4e-7


def test_deltas_of_very_different_sizes():
    """Pixel weights from 2^-60 to 1 within one image, and the same 2^-80 times as large, against 64 bits, every map by itself."""
    layers, patch, params, image, labels = case(3, 60, 64, 200, hidden=128)
    rng = np.random.default_rng(5)
    pixw = (2.0 ** rng.integers(-60, 1, labels.shape)).astype(np.float32)
    want = gradient64(layers, patch, params, image, labels, pixw)[0]
    for scale in (1.0, 2.0 ** -80):
        got = gradient(layers, patch, params, image, labels, pixw * np.float32(scale))[0] / scale
        assert np.isfinite(got).all()
        assert close_layers(got, want, layers, patch) <= bound(layers, patch)
        assert far_maps(got, want, layers, patch, [(0, "out", i) for i in range(60)] + [(1, "out", i) for i in range(64)]) <= 2 * bound(layers, patch)


def sums(side, low=0, spoil=None):
    """Second layer's outputs of sums of 64 side^2 products whose root of squares is about 8, of the library's own activations (`low`: a logistic net whose first layer's biases are
    that), at places where the squashing function is near its middle: the distance of the sums from those in 64 bits over the products' root of squares, rms."""
    layers, patch = ((C, 64, 3), (C, 40, side), (FC, 8, 0), (FC, 2, 0)), side + 4
    net = mpcnn.Net(layers, 1, patch)
    net.set_activation("logistic" if low else "tanh")
    rng = np.random.default_rng(side)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, patch + 60, patch + 71)).astype(np.float32)).cuda()
    params = rng.uniform(-0.7, 0.7, net.param_count).astype(np.float32)
    if low:
        params[576:640] = low
    second = params[640:640 + 40 * 64 * side * side]
    second *= np.float32((8 / 0.7 / side / 8 * 3) * (np.exp(-low) if low else 1))
    if spoil is not None:
        second[39 * 64 * side * side] = spoil
    y, pre, _, spread = (v[..., :39] for v in activations(net, layers, image, params))
    forward = [line for line in net.plan_describe(1, patch + 60, patch + 71, True).splitlines() if "forward: " in line][1]
    net.close()
    assert "or two of fp16" in forward, forward
    at = np.abs(pre) < 0.5
    assert at.sum() > 1000
    if low:
        y = np.log(y[at].astype(np.float64)) - np.log1p(-y[at].astype(np.float64))
    else:
        y = np.arctanh(y[at].astype(np.float64))
    return float(np.sqrt(((y - pre[at]) ** 2).mean() / (spread[at] ** 2).mean()))


@pytest.mark.parametrize("side", [5, 7, 11])
def test_sums_in_two_parts(side):
    """1600 to 7744 products.  Two parts lose 7.5e-8 of a sum (rms, the last bits and x1 y1); a run's roundings and the total's bring 5e-8 to 9e-8 (kernels_conv_parts.hpp measures 1.25e-7 together for 1600); half as
    much again is allowed.  Three parts are rounded in every step, and are taken where a weight (of another map) is infinite: other sums, and worse ones where the steps are 484."""
    two, three = sums(side), sums(side, spoil=np.inf)
    print("rms error of sums of %d products: two parts %.2e, three %.2e" % (64 * side * side, two, three), flush=True)
    assert two <= 1.7e-7 and two != three
    assert side < 11 or two < 0.8 * three


@pytest.mark.parametrize("low", [-3, -9, -12, -16, -20])
def test_small_logistic_outputs_under_large_weights(low):
    """A logistic output keeps its precision however small it is, and weights may make much of it: maps at 2^-4 under weights of up to 12 (two parts) and at 2^-13 to 2^-29 under weights of as much more
    (three).  As fp32 additions (above)."""
    assert sums(5, low=low) <= np.sqrt(1600 / 3) * 2.0 ** -24


def test_data_gradients_in_two_parts():
    """Bias gradients over the root of the deltas' squares, a pool-free net, 8000 positions: 4.4e-7 to 5.4e-7 with two parts, whose instructions are half as many, 1.25e-6 to 1.55e-6 with three:
    so these are two parts' sums."""
    layers, patch, H, W = ((C, 32, 5), (C, 64, 5), (C, 64, 3), (FC, 100, 0), (FC, 2, 0)), 14, 96, 110
    rng = np.random.default_rng(0)
    image = rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)
    labels = rng.integers(0, 2, (1, H, W)).astype(np.int32)
    net = mpcnn.Net(layers, 1, patch)
    params = rng.uniform(-0.05, 0.05, net.param_count).astype(np.float32)
    net.close()
    got, plan = gradient(layers, patch, params, image, labels)
    assert len([line for line in plan.splitlines() if "data gradient: " in line and "or two of fp16" in line]) == 3, plan
    want, deltas = gradient64(layers, patch, params, image, labels)
    ratios = [np.linalg.norm(got[at] - want[at]) / size for at, size in deltas[:3]]
    print("error of the bias gradients over the root of the deltas' squares:", " ".join("%.2e" % r for r in ratios), flush=True)
    assert max(ratios) <= 9e-7


# bf16 storage, eight tiles per wave (only where maps are large, never by a tiling hint): nets whose layers reach every such instance in both directions
WIDE_MAPS = [((C, 64, 3), (C, 64, 3), (C, 128, 3), (C, 64, 3)), ((C, 32, 3), (C, 128, 5), (C, 32, 5)), ((C, 64, 3), (C, 64, 5), (C, 64, 5)),
             ((C, 128, 3), (C, 128, 2), (C, 200, 2), (C, 128, 2))]
# channel counts 4 mod 8 (half an octet of the halo is another position's, stores of four channels), and a rectangular filter behind a pool of 2 x 3
WIDE_RAGGED = [(((C, 60, 3), (C, 100, 3), (C, 36, 3), (C, 60, 3), (FC, 8, 0), (FC, 2, 0)), 10), (((C, 60, 3), (MP, 0, 2, 3), (FC, 100, 0), (FC, 8, 0), (FC, 2, 0)), 8)]


def test_eight_tiles_per_wave_give_the_same_bits():
    """Against narrower tiles (a hint), which are held against the oracle: every sum is taken in the same order.  Both sides of a
    ragged map, channel counts that leave a tile empty (200 of 256) included."""
    wide, got = set(), set()
    text = open(os.path.join(os.path.dirname(mpcnn.__file__), "csrc", "launchers.hpp")).read()
    for f in re.findall(r"X\((\d+), (\d+), (\d+), (\d+), (\d+)\)", text[text.index("#define MPCNN_PARTS1_WIDE("):].split("#define", 2)[1]):
        wide.add(tuple(int(v) for v in f))
    assert wide
    for convs in WIDE_MAPS:
        layers = convs + ((FC, 8, 0), (FC, 2, 0))
        patch = sum(k - 1 for _, _, k in convs) + 2
        H, W = patch + 840, patch + 930
        net = mpcnn.Net(layers, 1, patch, mpcnn.BF16)
        rng = np.random.default_rng(patch)
        params, ci = [], 1
        for kind, m, k in layers:
            f = k if kind == C else (2 if m == 8 else 1)
            params.append(rng.uniform(-1, 1, m * ci * f * f + m) * 1.5 / np.sqrt(ci * f * f))
            ci = m
        net.set_params(np.concatenate(params).astype(np.float32))
        image = torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda()
        labels = torch.from_numpy(rng.integers(0, 2, (1, H, W)).astype(np.int32)).cuda()
        out = []
        for hint in ((0, 0), (4, 2)):
            net.set_conv_tiling(*hint)
            here = reached(net.plan_describe(1, H, W, True)) if hint == (0, 0) else set()
            got |= {r for r in here if r[1] in wide}
            probs = torch.empty((1, 2, H - patch + 1, W - patch + 1), device="cuda")
            net.seg_backward(image, labels, probs=probs)
            out.append((probs.cpu().numpy(), net.get_grads()))
        net.close()
        assert np.isfinite(out[0][1]).all() and np.any(out[0][1])
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]), convs
    assert got == {(d, i) for d in ("forward", "data gradient") for i in wide}, got
    for layers, patch in WIDE_RAGGED:
        H, W = patch + 840, patch + 930
        net = mpcnn.Net(layers, 1, patch, mpcnn.BF16)
        rng = np.random.default_rng(patch)
        net.set_params(rng.uniform(-0.1, 0.1, net.param_count).astype(np.float32))
        image = torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda()
        labels = torch.from_numpy(rng.integers(0, 2, (1, H, W)).astype(np.int32)).cuda()
        out = []
        for hint in ((0, 0), (4, 2)):
            net.set_conv_tiling(*hint)
            here = {d for d, i in reached(net.plan_describe(1, H, W, True)) if i in wide}
            assert here == ({"forward", "data gradient"} if hint == (0, 0) else set()), net.plan_describe(1, H, W, True)
            probs = torch.empty((1, 2, H - patch + 1, W - patch + 1), device="cuda")
            net.seg_backward(image, labels, probs=probs)
            out.append((probs.cpu().numpy(), net.get_grads()))
        net.close()
        assert np.isfinite(out[0][1]).all() and np.any(out[0][1])
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]), layers


# bf16 storage, layers behind the first.  Transposing reads: deltas whose last item has four channels.  One part per number: maps and channels 4 mod 8, a plane and half a
# unit past one, several groups of workgroups, filter sides 1 to 7
BF16_WGRAD = [(64, 100, 3, "tr"), (32, 36, 5, "tr"), (96, 140, 2, "tr"), (12, 28, 7, "one"), (16, 32, 5, "one"), (40, 100, 3, "one"), (64, 32, 3, "one"),
              (8, 48, 7, "bm"), (8, 32, 7, "one"), (36, 260, 1, "one"), (100, 36, 3, "one"), (48, 120, 5, "one"),
              (80, 32, (3, 2), "one"), (40, 100, (3, 2), "one")]      # (behind a pool of 2 x 3)
KERNEL = {"tr": "transposing reads", "one": "one part per number", "bm": "result tiles"}


@pytest.mark.parametrize("cin,cout,k,kernel", BF16_WGRAD)
def test_bf16_weight_gradient(cin, cout, k, kernel):
    """Deltas that are known exactly: the classes' biases saturate the softmax, so the last deltas are 0 or 1 and the layer's are a power of two
    times 1 - y y, rounded once.  Products of bf16 numbers are exact in fp32; an instruction adds 16 of them with two roundings (one of them to below), eight waves and
    every slab's sum is added once, so a gradient is off by at most (2 x instructions of a slab + 8 + slabs) 2^-23 of its products' absolute sum; one
    position that is missing or counted twice moves all gradients of its channel, by 1 / 17000 of that sum."""
    rect = isinstance(k, tuple)
    layers, patch = (((C, cin, 3), (MP, 0, 2, 3), (FC, cout, 0), (FC, 2, 0)), 8) if rect else (((C, cin, 3), (C, cout, k), (FC, 2, 0)), k + 2)
    (k, k2), (d, d2) = (k, (2, 3)) if rect else ((k, k), (1, 1))
    H, W = patch + 120, patch + 141
    net = mpcnn.Net(layers, 1, patch, mpcnn.BF16)
    plan = net.plan_describe(1, H, W, True)
    assert KERNEL[kernel] in [line for line in plan.splitlines() if "weight gradient" in line][1]
    r, c, slabs, tiles = [int(v) for v in re.findall(r"weight gradient: bf16 .*MFMA, .* tile (\d+) x (\d+).*, \d+ tiles in (\d+) slabs of (\d+)", plan)[-1]]
    rng = np.random.default_rng(cin)
    params = rng.uniform(-0.1, 0.1, net.param_count).astype(np.float32)
    w = np.zeros((2, cout), np.float32)
    w[0] = rng.choice([-1.0, 1.0], cout) * 2.0 ** -rng.integers(4, 7, cout)
    params[-2 * cout - 2:-2] = w.ravel()
    params[-2:] = 1000, -1000
    labels = rng.integers(0, 2, (1, H, W)).astype(np.int32)
    net.set_params(params)
    net.seg_backward(torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda(), torch.from_numpy(labels).cuda())
    got = net.get_grads().astype(np.float64)
    x, y = (torch.from_numpy(net.get_activation(1, H, W, i)[0]).double() for i in ((1, 2) if rect else (0, 1)))
    net.close()
    R, Q = y.shape[:2]
    at = (patch - 1) // 2
    t = torch.from_numpy(labels[0, at:at + R, at:at + Q]).double()[..., None]
    dy = (t * torch.from_numpy(w[0]).double() * (1 - y * y)).float().bfloat16().double().reshape(-1, cout)
    part = lambda u, v: x[u * d:u * d + R, v * d2:v * d2 + Q].reshape(-1, cin)
    taps = [(u, v) for u in range(k) for v in range(k2)]
    want, mass = (torch.stack([f(dy).t().contiguous() @ f(part(u, v)) for u, v in taps], -1).flatten().numpy() for f in (lambda z: z, torch.abs))
    first = cin * 9 + cin
    bound = (2 * tiles * r * -(-c // 16) + slabs + 8) * 2.0 ** -23
    assert (np.abs(got[first:first + want.size] - want) <= bound * mass).all()
    assert bound < 1.0 / (R * Q) and np.any(want)
    bias = got[first + want.size:first + want.size + cout] - dy.sum(0).numpy()
    assert (np.abs(bias) <= (R * Q) * 2.0 ** -24 * dy.abs().sum(0).numpy()).all()


# fp32 storage: chains of positions on either side of the line from which two parts are taken
CHAINS = [(32, 64, 5, 58, 61, False), (16, 36, 5, 100, 110, False), (64, 128, 3, 200, 190, True), (20, 44, 4, 420, 390, True)]


@pytest.mark.parametrize("cin,cout,k,R,Q,two", CHAINS)
def test_fp32_weight_gradient(cin, cout, k, R, Q, two):
    """Deltas that are known exactly: saturated classes, and a layer whose weights are so small that all slopes are 1.  A chunk of 16 positions is six instructions
    of two roundings and a truncation each at most, so a gradient is off by at most (18 x chunks of a wave + 8 + slabs) 2^-24 of its products' absolute sum, and by
    2^-22 for what two parts leave out of a product."""
    layers, patch = ((C, cin, 3), (C, cout, k), (FC, 2, 0)), k + 2
    H, W = R + patch - 1, Q + patch - 1
    net = mpcnn.Net(layers, 1, patch)
    line = [line for line in net.plan_describe(1, H, W, True).splitlines() if "weight gradient" in line][1]
    assert "three parts per number" in line and ("or two of fp16" in line) == two, line
    wk, r, c, slabs, tiles = [int(v) for v in re.search(r"x (\d+) waves .* tile (\d+) x (\d+), \d+ tiles in (\d+) slabs of (\d+)", line).groups()]
    rng = np.random.default_rng(cin)
    params = rng.uniform(-0.7, 0.7, net.param_count).astype(np.float32)
    first = cin * 9 + cin
    n = cout * cin * k * k
    params[first:first + n + cout] *= 1e-12
    w = np.zeros((2, cout), np.float32)
    w[0] = rng.uniform(-1, 1, cout)
    params[-2 * cout - 2:-2] = w.ravel()
    params[-2:] = 1000, -1000
    labels = rng.integers(0, 2, (1, H, W)).astype(np.int32)
    net.set_params(params)
    net.seg_backward(torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda(), torch.from_numpy(labels).cuda())
    got = net.get_grads().astype(np.float64)[first:first + n]
    x = torch.from_numpy(net.get_activation(1, H, W, 0)[0]).double()
    net.close()
    at = (patch - 1) // 2
    dy = (torch.from_numpy(labels[0, at:at + R, at:at + Q]).double()[..., None] * torch.from_numpy(w[0]).double()).reshape(-1, cout)
    taps = [x[u:u + R, v:v + Q].reshape(-1, cin) for u in range(k) for v in range(k)]
    want, mass = (torch.stack([f(dy).t().contiguous() @ f(t) for t in taps], -1).flatten().numpy() for f in (lambda z: z, torch.abs))
    assert (np.abs(got - want) <= ((18 * tiles * r * (c // 16) // wk + 8 + slabs) * 2.0 ** -24 + 2.0 ** -22) * mass).all()
    # two parts in the 2-norm: 5e-8, measured over chains of 144 to 640 positions, and twice that
    assert np.linalg.norm(got - want) <= 1e-7 * np.linalg.norm(want)


def known_deltas(cin, cout, k, R, Q, class_weights, bias=None, pixw=None, logistic=False, own_bias=None):
    """A layer's weight gradient [maps, inputs, taps], the same in 64 bits, and its plan, from deltas that are known exactly: saturated classes, and a layer whose weights are so
    small that all slopes are 1 (logistic: 1/4, or that of the maps' own biases).  The inputs are the library's own."""
    layers, patch = ((C, cin, 3), (C, cout, k), (FC, 2, 0)), k + 2
    H, W = R + patch - 1, Q + patch - 1
    net = mpcnn.Net(layers, 1, patch)
    net.set_activation("logistic" if logistic else "tanh")
    rng = np.random.default_rng(cin)
    params = rng.uniform(-0.7, 0.7, net.param_count).astype(np.float32)
    first = cin * 9 + cin
    n = cout * cin * k * k
    if bias is not None:
        params[cin * 9:first] = bias
    params[first:first + n + cout] *= 1e-12
    if own_bias is not None:
        params[first + n:first + n + cout] = own_bias
    w = np.zeros((2, cout), np.float32)
    w[0] = class_weights
    params[-2 * cout - 2:-2] = w.ravel()
    params[-2:] = 1000, -1000
    labels = rng.integers(0, 2, (1, H, W)).astype(np.int32)
    net.set_params(params)
    plan = [line for line in net.plan_describe(1, H, W, True).splitlines() if "weight gradient" in line][1]
    net.seg_backward(torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda(), torch.from_numpy(labels).cuda(),
                     pixw=None if pixw is None else torch.from_numpy(pixw).cuda())
    got = net.get_grads().astype(np.float64)[first:first + n].reshape(cout, cin, k * k)
    x, h = (torch.from_numpy(net.get_activation(1, H, W, layer)[0]).double() for layer in (0, 1))
    net.close()
    at = (patch - 1) // 2
    slope = (h * (1 - h).float().double()).float().double() if logistic else 1.0     # (two fp32 operations)
    t = torch.from_numpy(labels[0, at:at + R, at:at + Q]).double()
    if pixw is not None:
        t = t * torch.from_numpy(pixw[0, at:at + R, at:at + Q]).double()
    dy = (t[..., None] * (torch.from_numpy(w[0]).double() * slope).float().double()).reshape(-1, cout)
    want = torch.stack([dy.t().contiguous() @ x[u:u + R, v:v + Q].reshape(-1, cin) for u in range(k) for v in range(k)], -1).numpy()
    return got, want, plan


def by_map(got, want, axes):
    return np.sqrt(((got - want) ** 2).sum(axes)) / np.sqrt((want ** 2).sum(axes))


# Two parts of a delta are off by 2^-23 of it at most, here the same for all positions of a map whose deltas are 0 or one number; activations, products left
# out and sums bring 5e-8 in the 2-norm (measured over chains of 144 to 640 positions, csrc/mpcnn.hip, kHalfChain)
MAP_BOUND = 2.0 ** -23 + 5e-8
WGRAD = (64, 128, 3, 200, 190)


NEAR = [9, 13, 18, 20, 22, 25, 11, 12, 14, 15, 16, 17, 19, 21, 23, 24]


@pytest.mark.parametrize("shape,octaves", [(WGRAD, NEAR), ((20, 44, 4, 420, 390), NEAR), (WGRAD, [26, 30, 35, 40, 60, 100] + NEAR[:10])])
def test_weight_gradient_of_maps_far_below_the_others(shape, octaves):
    """Deltas of every eighth map 2^-9 to 2^-25 of the others', and to 2^-100 (the class layer's weights say so: three parts): each map's gradient as close to 64 bits as the others'."""
    rng = np.random.default_rng(1)
    w = rng.choice([-1.0, 1.0], shape[1]) * rng.uniform(0.5, 1, shape[1])
    w[::8] *= 2.0 ** -np.array(octaves[:len(w[::8])])
    got, want, plan = known_deltas(*shape, w)
    assert "or two of fp16" in plan, plan
    err = by_map(got, want, (1, 2))
    print("maps far below the others:", " ".join("%.1e" % e for e in err[::8]), "others:", "%.1e" % np.delete(err, np.s_[::8]).max(), flush=True)
    assert err.max() <= MAP_BOUND


def test_weight_gradient_of_maps_that_stand_out_in_few_positions():
    """Pixel weights of 2^-17 but for three positions of 1, and some maps 2^-10 of the others: deltas down to 2^-28 of the largest keep their bits.  One of
    the three stands in an accumulator for the rest of a slab, 10 chunks of six products with two roundings each: sqrt(120 / 3) 2^-24 besides."""
    rng = np.random.default_rng(2)
    w = rng.choice([-1.0, 1.0], 128) * rng.uniform(0.5, 1, 128)
    w[::8] *= 2.0 ** -10
    w[1] = 0
    pixw = np.full((1, 204, 194), 2.0 ** -17, np.float32)
    pixw[0, [40, 90, 177], [61, 33, 150]] = 1
    got, want, _ = known_deltas(*WGRAD, w, pixw=pixw)
    assert not got[1].any()
    keep = np.arange(128) != 1
    assert by_map(got[keep], want[keep], (1, 2)).max() <= MAP_BOUND + np.sqrt(40) * 2.0 ** -24


def test_weight_gradient_of_few_labels():
    """Deltas that are zero but in a corner."""
    pixw = np.zeros((1, 204, 194), np.float32)
    pixw[0, 150:155, 11:17] = 1
    got, want, _ = known_deltas(*WGRAD, np.linspace(0.1, 1, 128), pixw=pixw)
    assert by_map(got, want, (1, 2)).max() <= MAP_BOUND


@pytest.mark.parametrize("low", [False, True])
def test_weight_gradient_of_logistic_maps(low):
    """Logistic outputs keep their precision however small they are: maps of biases 0 to -60 (outputs down to 2^-87), every input map by itself."""
    bias = np.zeros(64)
    if low:
        bias[::4] = -np.array([4, 6, 8, 10, 12, 14, 16, 18, 20, 22, 24, 28, 32, 40, 50, 60])
    got, want, plan = known_deltas(*WGRAD, np.random.default_rng(3).uniform(0.2, 1, 128), bias=bias, logistic=True)
    assert "or two of fp16" in plan, plan
    err = by_map(got, want, (0, 2))
    print("input maps:", " ".join("%.1e" % e for e in err[::4]), flush=True)
    assert err.max() <= MAP_BOUND and by_map(got, want, (1, 2)).max() <= MAP_BOUND


def test_weight_gradient_below_logistic_units_that_are_off():
    """Logistic units at biases of -10 to -60: slopes, and so deltas, down to 2^-87, every map by itself."""
    own = np.zeros(128)
    own[::8] = -np.array([4, 6, 8, 10, 12, 14, 16, 18, 20, 22, 24, 28, 32, 40, 50, 60])
    got, want, _ = known_deltas(*WGRAD, np.random.default_rng(4).uniform(0.2, 1, 128), logistic=True, own_bias=own)
    err = by_map(got, want, (1, 2))
    print("maps of units that are off:", " ".join("%.1e" % e for e in err[::8]), flush=True)
    assert err.max() <= MAP_BOUND


@pytest.mark.parametrize("logistic", [False, True])
def test_few_positions_with_large_deltas_take_no_longer(logistic):
    """A net that is sure of nearly all its labels (class weights 1000 times as large, 3 in 10 000 labels wrong): its weight gradients, microseconds, against those of an unsure one."""
    layers, patch = ((C, 64, 3), (C, 64, 3), (C, 64, 3), (FC, 128, 0), (FC, 2, 0)), 9
    H, W = 600, 610
    net = mpcnn.Net(layers, 1, patch)
    net.set_activation("logistic" if logistic else "tanh")
    rng = np.random.default_rng(7)
    params = (rng.uniform(-1, 1, net.param_count) * 0.05).astype(np.float32)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda()
    took = []
    for factor in (1, 1000):
        params[-2 * 128 - 2:] *= factor
        net.set_params(params)
        label = net.seg_forward(image, torch.empty((1, 2, H - patch + 1, W - patch + 1), device="cuda"))[0].argmax(0).cpu().numpy()
        wrong = rng.uniform(size=label.shape) < 3e-4
        labels = np.zeros((1, H, W), np.int32)
        at = (patch - 1) // 2
        labels[0, at:at + label.shape[0], at:at + label.shape[1]] = np.where(wrong, 1 - label, label)
        labels = torch.from_numpy(labels).cuda()
        net.seg_backward(image, labels)
        net.profile_enable(True)
        for _ in range(5):
            net.seg_backward(image, labels)
        took.append(sum(1e3 * r["ms_total"] / r["launches"] for r in net.profile_read() if r["name"] == "wgrad_parts"))
        net.profile_enable(False)
    net.close()
    print("weight gradients of an unsure and a sure net: %.0f, %.0f us" % tuple(took), flush=True)
    assert took[1] <= 1.25 * took[0]
