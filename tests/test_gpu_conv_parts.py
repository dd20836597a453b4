"""Convolutions (either storage type) and fp32 weight gradients on the bf16 matrix instruction, fp32 numbers as sums of
bf16 parts (csrc/kernels_conv_parts.hpp, csrc/kernels_wgrad_parts.hpp): shapes at the edges of their tiles, channel blocks and groups against the oracle,
numbers that have no parts, and the distance from 64-bit sums."""
import os
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1302_1690_amd import mpcnn, workloads as wl
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
C, MP, FC = wl.C, wl.MP, wl.FC

# channel counts 4 mod 8, one past a block of 16 / 32 channels, one past a group of 4 channel tiles; filters of
# side 1, 2, 3, 5; maps of a few positions up to several ragged tiles
EDGES = [
    ("quads", ((C, 12, 3), (MP, 0, 2), (C, 20, 2), (FC, 36, 0), (FC, 3, 0)), 14, 31, 38),
    ("past_a_group", ((C, 8, 3), (C, 132, 3), (MP, 0, 2), (C, 36, 2), (FC, 8, 0), (FC, 2, 0)), 14, 40, 33),
    ("units", ((C, 16, 3), (MP, 0, 2), (FC, 44, 0), (FC, 10, 0), (FC, 9, 0), (FC, 2, 0)), 4, 37, 41),
    ("wide_filter", ((C, 40, 2), (C, 17, 5), (MP, 0, 3), (C, 24, 2), (FC, 33, 0), (FC, 2, 0)), 12, 52, 47),
    # weight gradient: 8 and 7 column tiles, 27 and 58 units, several groups of workgroups
    ("groups", ((C, 48, 3), (C, 232, 3), (MP, 0, 2), (C, 200, 2), (FC, 12, 0), (FC, 2, 0)), 14, 34, 52),
    ("one_position", ((C, 16, 3), (MP, 0, 2), (C, 32, 3), (FC, 64, 0), (FC, 2, 0)), 10, 10, 10),
    # the first and the third on maps large enough for the weight gradient in three parts
    ("quads_many", ((C, 12, 3), (MP, 0, 2), (C, 20, 2), (FC, 36, 0), (FC, 3, 0)), 14, 151, 158),
    ("units_many", ((C, 16, 3), (MP, 0, 2), (FC, 44, 0), (FC, 10, 0), (FC, 9, 0), (FC, 2, 0)), 4, 117, 131),
]


# filters whose halo is taken in blocks of fewer rows: the whole patch left of a layer (spacing 1 and 2), several channel blocks, a last
# block of one row, 8 channels in a block of 16
LARGE = [
    ("rows_of_26", ((C, 16, 3), (C, 12, 26), (MP, 0, 2), (FC, 8, 0), (FC, 2, 0)), 30, 47, 52),
    ("rows_of_33", ((C, 20, 2), (C, 36, 33), (FC, 8, 0), (FC, 2, 0)), 35, 50, 46),
    ("fc_over_30", ((C, 8, 5), (MP, 0, 2), (FC, 32, 0), (FC, 2, 0)), 64, 77, 82),
    ("rows_of_45", ((C, 8, 3), (C, 8, 45), (FC, 8, 0), (FC, 2, 0)), 49, 58, 61),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name,layers,patch,height,width", EDGES + LARGE, ids=[e[0] for e in EDGES + LARGE])
def test_tile_and_channel_edges(name, layers, patch, height, width, dtype):
    full_parity(wl.Workload("parts_" + name, layers, patch, 1, layers[-1][1], 2, height, width, 0.2, "ellipses", dtype=dtype,
                            seed_image=1141, seed_label=2141, seed_param=3141), with_pixw=True)


def activations(net, layers, image, params):
    """The library's output of the second layer and, from its first layer's, the sums behind it in 64 bits: the
    sum, the sum of the products' sizes, and the root of the sum of their squares."""
    B, _, H, W = image.shape
    net.set_params(params)
    net.seg_backward(image, torch.zeros((B, H, W), dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    x, y = net.get_activation(B, H, W, 0), net.get_activation(B, H, W, 1)
    (_, m0, k0), (_, m1, k1) = layers[0], layers[1]
    at = m0 * k0 * k0 + m0
    w = torch.from_numpy(params[at:at + m1 * m0 * k1 * k1].reshape(m1, m0, k1, k1)).double()
    b = torch.from_numpy(params[at + w.numel():at + w.numel() + m1]).double()
    x64 = torch.from_numpy(x).double().permute(0, 3, 1, 2)
    conv = torch.nn.functional.conv2d
    sums = (conv(x64, w, b), conv(x64.abs(), w.abs(), b.abs()), conv(x64 * x64, w * w, b * b).sqrt())
    return (y,) + tuple(t.permute(0, 2, 3, 1).numpy() for t in sums)


def test_sums_are_as_close_as_fp32_ones():
    """tanh of a sum of 576 products in 36 steps of one instruction for the leading products and five for those 2^-8 as large,
    two roundings each: 72 (1 + 5 / 256) of them count.  One moves the running sum by at most 2^-24
    of its size, so all by at most 74 2^-24 of the products' absolute sum; in the root mean square, by
    sqrt(74 / 3) 2^-24 of the running sum's root mean square, which random signs keep below the root of the sum of
    squares.  What is left out of a product is at most 2^-24 of it (2^-26 rms); the hardware exp2 and reciprocal bring 2e-7 (1.2e-7 rms).
    576 fp32 additions one after the other would be allowed sqrt(576 / 3)."""
    layers = ((C, 64, 3), (C, 96, 3), (FC, 8, 0), (FC, 2, 0))
    net = mpcnn.Net(layers, 1, 6)
    rng = np.random.default_rng(5)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, 40, 43)).astype(np.float32)).cuda()
    params = (0.05 * rng.standard_normal(net.param_count) * np.exp(rng.standard_normal(net.param_count))).astype(np.float32)
    y, pre, mass, spread = activations(net, layers, image, params)
    err = np.abs(y - np.tanh(pre))
    assert (err <= (74 + 1) * 2.0 ** -24 * mass + 2e-7).all()
    rms = lambda v: np.sqrt((v ** 2).mean())
    assert rms(err) <= np.hypot(np.hypot(np.sqrt(74 / 3) * 2.0 ** -24, 2.0 ** -26) * rms(spread), 1.2e-7)
    net.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.395e38])
def test_numbers_without_parts(value):
    """Infinities, NaN and numbers above the largest bf16 in a layer's weights reach the outputs that use
    them as fp32 arithmetic has it, and no others."""
    layers = ((C, 16, 3), (C, 40, 3), (FC, 8, 0), (FC, 2, 0))
    net = mpcnn.Net(layers, 1, 6)
    rng = np.random.default_rng(6)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, 30, 27)).astype(np.float32)).cuda()
    params = rng.uniform(-0.2, 0.2, net.param_count).astype(np.float32)
    at = 16 * 9 + 16
    params[at + (37 * 16 + 5) * 9 + 4] = value           # map 37, channel 5, middle tap
    y, pre, _, _ = activations(net, layers, image, params)
    want = np.tanh(pre)
    assert np.array_equal(np.isnan(y), np.isnan(want))
    ok = ~np.isnan(want)
    assert np.isfinite(y[ok]).all() and np.abs(y[ok] - want[ok]).max() <= 1e-6
    net.close()


def test_delta_that_is_not_finite_stays_where_it_is():
    """A pixel weight of NaN: the deltas of the positions its patch covers are NaN, every activation and the other
    pixels' probabilities are what they were."""
    layers = ((C, 16, 3), (C, 32, 3), (FC, 24, 0), (FC, 2, 0))
    net = mpcnn.Net(layers, 1, 6)
    rng = np.random.default_rng(7)
    B, H, W = 1, 24, 29
    image = torch.from_numpy(rng.uniform(0, 1, (B, 1, H, W)).astype(np.float32)).cuda()
    labels = torch.zeros((B, H, W), dtype=torch.int32, device="cuda")
    net.set_params(rng.uniform(-0.2, 0.2, net.param_count).astype(np.float32))
    out = []
    for bad in (False, True):
        pixw = torch.ones((B, H, W), device="cuda")
        if bad:
            pixw[0, 10, 12] = float("nan")
        probs = torch.empty((B, 2, H - 5, W - 5), device="cuda")
        net.seg_backward(image, labels, pixw=pixw, probs=probs)
        out.append((probs.cpu().numpy(), net.get_grads()))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.isfinite(out[0][1]).all() and np.isnan(out[1][1]).all()
    net.close()


def test_sums_are_not_off_to_one_side():
    """Bias gradients sum deltas over 8000 positions whose signs are random: what rounding leaves of each sums to sqrt(8000) of
    it, an offset to one side to 8000 of it.  Layers without pools (no ties), labels at random; the 64-bit
    values from autograd.  Allowed is what fp32 additions may leave, two products each: a delta is the sum of up to 1600 products, in the root mean
    square off by sqrt(800 / 3) 2^-24 of the running sum's root mean square, at most the sum's own: 1.0e-6.  Each of the two convolutions
    below adds as much again (so sqrt(3) of it), and the positions' errors, independent of each other, their root of squares.  Twice that is
    allowed; with one accumulator for all six products, whose results are 8e-8 too low, the error is 1e-5."""
    layers = ((C, 32, 5), (C, 64, 5), (C, 64, 3), (FC, 100, 0), (FC, 2, 0))
    patch, H, W = 14, 96, 110
    net = mpcnn.Net(layers, 1, patch)
    ratios = []
    for seed in range(2):
        rng = np.random.default_rng(seed)
        image = torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32))
        labels = torch.from_numpy(rng.integers(0, 2, (1, H, W)).astype(np.int32))
        params = rng.uniform(-0.05, 0.05, net.param_count).astype(np.float32)
        net.set_params(params)
        net.seg_backward(image.cuda(), labels.cuda())
        grads = net.get_grads().astype(np.float64)
        x, at, side, ci, fc, pre, places = image.double(), 0, patch, 1, False, [], []
        for i, (kind, m, k) in enumerate(layers):
            k = k if kind == C else (1 if fc else side)
            w = torch.from_numpy(params[at:at + m * ci * k * k].astype(np.float64).reshape(m, ci, k, k))
            at += w.numel()
            x = torch.nn.functional.conv2d(x, w, torch.from_numpy(params[at:at + m].astype(np.float64)))
            if i == 0:
                x.requires_grad_()
            else:
                x.retain_grad()
            pre.append(x)
            places.append(slice(at, at + m))
            at += m
            if i < len(layers) - 1:
                x = torch.tanh(x)
            side, ci, fc = (side - k + 1 if kind == C else 1), m, fc or kind == FC
        c = (patch - 1) // 2
        target = labels[:, c:c + x.shape[2], c:c + x.shape[3]].long()
        torch.nn.functional.cross_entropy(x, target, reduction="sum").backward()
        for layer in range(3):
            delta = pre[layer].grad[0]                     # [maps, rows, columns]
            off = grads[places[layer]] - delta.sum((1, 2)).numpy()
            ratios.append(np.sqrt((off ** 2).sum() / float((delta ** 2).sum())))
    print("error of the bias gradients over the root of the deltas' squares:", " ".join("%.2e" % r for r in ratios), flush=True)
    net.close()
    assert max(ratios) <= 2 * np.sqrt(3) * np.sqrt(800 / 3) * 2.0 ** -24


def test_weight_gradients_are_not_off_to_one_side():
    """A weight gradient of 32 -> 64 channels, 5 x 5, summed over a million positions in many slabs, against 64-bit sums of the library's own
    activations and the deltas that follow from them.  All labels are one class, so that a slab's sums are large and keep their
    sign.  The errors of 64 output channels, each with deltas of its own, average to an eighth of their size where none leans
    to one side; four times that is allowed.  With every slab's results a little too low the average is 0.57 of their size."""
    ci, co, k, side = 32, 64, 5, 1024
    net = mpcnn.Net(((C, ci, 3), (C, co, k), (FC, 2, 0)), 1, k + 2)
    rng = np.random.default_rng(3)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, side, side)).astype(np.float32)).cuda()
    params = (rng.uniform(-1, 1, net.param_count) * 0.1).astype(np.float32)
    net.set_params(params)
    net.seg_backward(image, torch.zeros((1, side, side), dtype=torch.int32, device="cuda"))
    grads = net.get_grads().astype(np.float64)
    x, h = (torch.from_numpy(net.get_activation(1, side, side, l)[0]).cuda() for l in (0, 1))
    net.close()
    rows, cols = h.shape[:2]
    h = h.reshape(-1, co).double()
    first = ci * 9 + ci
    last = first + co * ci * k * k + co
    w = torch.from_numpy(params[last:last + 2 * co].reshape(2, co)).cuda().double()
    b = torch.from_numpy(params[last + 2 * co:]).cuda().double()
    d = torch.softmax(torch.mm(h, w.t().contiguous()) + b, 1)
    d[:, 0] -= 1
    d = (torch.mm(d, w) * (1 - h * h)).t().contiguous()
    want = torch.stack([torch.mm(d, x[u:u + rows, v:v + cols].reshape(-1, ci).double()) for u in range(k) for v in range(k)], 2)
    err = grads[first:last - co] - want.cpu().numpy().ravel()
    mean, rms = err.mean(), np.sqrt((err ** 2).mean())
    print("weight gradient: error %.2e of its size, on average %.2f of that to one side" % (np.linalg.norm(err) / np.linalg.norm(want.cpu().numpy()), mean / rms), flush=True)
    assert abs(mean) <= 0.5 * rms


def gradients(layers, patch, params, pixw=None):
    net = mpcnn.Net(layers, 1, patch)
    rng = np.random.default_rng(11)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, 72, 71)).astype(np.float32)).cuda()
    labels = torch.from_numpy(rng.integers(0, 2, (1, 72, 71)).astype(np.int32)).cuda()
    net.set_params(params)
    net.seg_backward(image, labels, pixw=None if pixw is None else torch.full((1, 72, 71), pixw, device="cuda"))
    grads = net.get_grads().astype(np.float64)
    net.close()
    return grads


SMALL = ((C, 16, 3), (C, 40, 3), (FC, 24, 0), (FC, 2, 0))   # patch 8, no pools


def close_layers(got, want, layers, patch):
    """Largest relative distance (2-norm) of a layer's gradient."""
    side, ci, at, worst, fc = patch, 1, 0, 0.0, False
    for kind, m, k in layers:
        k = k if kind == C else (1 if fc else side)
        n = m * ci * k * k + m
        worst = max(worst, np.linalg.norm(got[at:at + n] - want[at:at + n]) / np.linalg.norm(want[at:at + n]))
        at, ci, fc, side = at + n, m, fc or kind == FC, side - k + 1
    return worst


def test_small_numbers_keep_their_bits():
    """Everything behind the forward pass is linear in the pixel weights, and the delta below a layer in its weights: made a
    power of two smaller, every fp32 operation rounds as before, until numbers are subnormal and off by 2^-150 each.
    Pixel weights of 2^-114: deltas from 2^-115 to 2^-125, of which 2^-133 (the last bit of bf16) would be 2^-18 to 2^-8.
    A gradient adds 4700 products of them, whose 2^-150 are below 2^-24 of the deltas' size each: 2^-20 allows for all."""
    rng = np.random.default_rng(12)
    params = rng.uniform(-0.2, 0.2, mpcnn.Net(SMALL, 1, 8).param_count).astype(np.float32)
    small = gradients(SMALL, 8, params, 2.0 ** -114)
    assert close_layers(small * 2.0 ** 114, gradients(SMALL, 8, params, 1.0), SMALL, 8) <= 2.0 ** -20
    # the second layer's weights at 2^-40 and 2^-114 of these: the layers above see its biases either way
    at = 16 * 9 + 16
    got = []
    for e in (-40, -114):
        p = params.copy()
        p[at:at + 40 * 16 * 9] *= np.float32(2.0 ** e)
        got.append(gradients(SMALL, 8, p)[:at] * 2.0 ** -e)
    assert np.linalg.norm(got[1] - got[0]) <= 2.0 ** -20 * np.linalg.norm(got[0])


WIDE = ((C, 48, 3), (C, 132, 3), (C, 72, 2), (FC, 40, 0), (FC, 2, 0))   # patch 8, no pools; several planes, taps and groups


def test_deltas_without_parts():
    """Pixel weights of 2^114: no delta has parts, so every element of the data gradients (borders included) and of the weight
    gradients is computed again with fp32 multiply-adds, and stays below the largest fp32 number.  They are 2^114 times those of
    pixel weights 1, whose sums are taken in another order: two sums of up to 4700 products, each off by
    sqrt(4700 / 3) 2^-24 of the running sum, 2.4e-6 each; 2^-17 allows twice that on both sides."""
    rng = np.random.default_rng(13)
    params = rng.uniform(-0.1, 0.1, mpcnn.Net(WIDE, 1, 8).param_count).astype(np.float32)
    big = gradients(WIDE, 8, params, 2.0 ** 114)
    assert np.isfinite(big).all()
    assert close_layers(big * 2.0 ** -114, gradients(WIDE, 8, params, 1.0), WIDE, 8) <= 2.0 ** -17


def test_weights_without_parts_in_the_data_gradient():
    """A weight that has no parts: its map is saturated, its delta 0 and 0 times the weight 0, so the deltas below are what they are
    without it: as far from those of a weight of 2^100 (which has parts, saturates as well) as the rounding of sums in another order (above)."""
    rng = np.random.default_rng(14)
    params = rng.uniform(-0.1, 0.1, mpcnn.Net(WIDE, 1, 8).param_count).astype(np.float32)
    at = 48 * 9 + 48 + 132 * 48 * 9 + 132 + (37 * 132 + 45) * 4 + 1   # third layer: map 37, channel 45, tap 1
    params[48 * 9 + 48 + 132 * 48 * 9 + 45] = 4.0                     # (channel 45 is nowhere near 0)
    got = []
    for value in (2.0 ** 100, 3.395e38):
        params[at] = value
        got.append(gradients(WIDE, 8, params))
    assert np.isfinite(got[0]).all() and np.isfinite(got[1]).all()
    assert close_layers(got[1], got[0], WIDE, 8) <= 2.0 ** -17


def test_a_net_that_diverged_is_not_slow():
    """Training steps with parameters that are all NaN, and with one infinite weight per layer, against finite ones: the sums that are not
    finite are computed again, which takes as long as a value, or as the few maps that need it (times before that was so:
    see the factor that is printed)."""
    cfg = wl.crop(wl.CONFIGS[3], 1, 330, 340)
    img, lab = wl.make_inputs(cfg)
    params = wl.make_params(cfg)
    image, labels = torch.from_numpy(img).cuda(), torch.from_numpy(lab).cuda()
    one = params.copy()
    for layer in (2, 4, 6):
        at = sum(m * ci * k * k + m for ci, m, k in wl_layers(cfg)[:layer // 2])
        one[at + 3] = np.inf
    ms = []
    for p in (params, np.full_like(params, np.nan), one):
        net = mpcnn.Net(cfg.layers, cfg.in_channels, cfg.patch)
        net.set_params(p)
        net.seg_backward(image, labels)
        torch.cuda.synchronize()
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            net.seg_backward(image, labels)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
        net.close()
    print("finite, NaN, one infinite weight per layer: %.2f, %.2f, %.2f ms (x %.2f, %.2f)" % (*ms, ms[1] / ms[0], ms[2] / ms[0]), flush=True)
    assert ms[1] <= 1.5 * ms[0] and ms[2] <= 20 * ms[0]


def wl_layers(cfg):
    """(inputs, maps, filter side) of the layers with parameters."""
    side, ci, fc, out = cfg.patch, cfg.in_channels, False, []
    for kind, m, k in cfg.layers:
        if kind == MP:
            side //= k
            continue
        k = k if kind == C else (1 if fc else side)
        out.append((ci, m, k))
        ci, fc, side = m, fc or kind == FC, side - k + 1
    return out


# channel counts that give every pair of block width (16, 32, 64, 128 input channels) and channel tiles (1, 2, 4, an odd number)
# in both directions
CHANNELS = [(16, 16, 64, 64, 32, 128, 128, 96), (16, 128, 64, 96, 32, 32, 64, 128, 32), (16, 96, 128, 16, 32, 64, 16)]
HINTS = {"f32": [(0, 0), (4, 1), (8, 2), (2, 1), (4, 2), (2, 2)], "bf16": [(0, 0), (8, 2), (16, 4), (4, 2), (2, 2), (4, 4)]}


def instances(dtype):
    """The tuples the library is built with, from its list."""
    text = open(os.path.join(os.path.dirname(mpcnn.__file__), "csrc", "launchers.hpp")).read()
    at = text.index("#define MPCNN_PARTS%d(" % (1 if dtype == "bf16" else 3))
    found = re.findall(r"X\((\d+), (\d+), (\d+), (\d+), (\d+)\)", text[at:text.index("#define", at + 8)])
    return {tuple(int(v) for v in f) for f in found}


def reached(plan):
    """(direction, (channels per block, waves along channels, along positions, tiles per wave along both)) of a plan's convolutions."""
    return {(m[1], (int(m[6]), int(m[2]), int(m[3]), int(m[4]), int(m[5])))
            for m in re.finditer(r"(forward|data gradient): bf16 MFMA.*?waves (\d) x (\d) of (\d) x (\d) tiles, (\d+) channels", plan)}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_every_instance_gives_the_same_bits(dtype):
    """Every instance the library is built with, in both directions: probabilities and gradients do not depend on which one runs, as every
    sum is taken in the same order (the planner's own choice is held against the oracle above)."""
    got = set()
    for channels in CHANNELS:
        # (narrower blocks than the channels allow: filters whose halo has no room for more)
        for k, size in ((3, 40), (11, 20)) if channels is CHANNELS[0] else ((3, 40),):
            layers = tuple((C, c, k) for c in channels) + ((FC, 8, 0), (FC, 2, 0))
            patch = len(channels) * (k - 1) + 2
            H, W = patch + size, patch + size + 7
            net = mpcnn.Net(layers, 1, patch, mpcnn.BF16 if dtype == "bf16" else mpcnn.F32)
            rng = np.random.default_rng(patch)
            scale = np.concatenate([np.full(m * ci * f * f + m, 1.5 / np.sqrt(m * f * f))
                                    for ci, m, f in zip((1,) + channels + (8,), channels + (8, 2), (k,) * len(channels) + (2, 1))])
            net.set_params((scale * rng.uniform(-1, 1, net.param_count)).astype(np.float32))
            image = torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda()
            labels = torch.from_numpy(rng.integers(0, 2, (1, H, W)).astype(np.int32)).cuda()
            first = None
            for hint in HINTS[dtype]:
                net.set_conv_tiling(*hint)
                got |= reached(net.plan_describe(1, H, W, True))
                probs = torch.empty((1, 2, H - patch + 1, W - patch + 1), device="cuda")
                net.seg_backward(image, labels, probs=probs)
                out = (probs.cpu().numpy(), net.get_grads())
                first = first or out
                assert np.isfinite(out[1]).all() and np.any(out[1])
                assert np.array_equal(out[0], first[0]) and np.array_equal(out[1], first[1]), (channels, k, hint)
            net.close()
    want = {(d, i) for d in ("forward", "data gradient") for i in instances(dtype)}
    assert got == want, sorted(want - got)
