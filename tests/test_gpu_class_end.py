"""The hidden layer that ends with the class layer (calls that keep nothing: probabilities, losses of a line search): the same bits as the training
pass, whose class layer is a launch of its own, for every instance of the kernel, odd channel counts, both losses and squashing functions, positions
of less than a tile, and sums that are not finite."""
import re
from pathlib import Path

import numpy as np
import pytest
import torch

from paper_1302_1690_amd import mpcnn, workloads as wl
from test_gpu_parity import full_parity

C, MP, FC = wl.C, wl.MP, wl.FC
pytestmark = pytest.mark.gpu
AT_END = "class layer: at the end of the layer below"


def check(layers, patch, B, H, W, dtype, loss, squash, seen=None, params=None, at_end=True):
    net = mpcnn.Net(layers, 1, patch, mpcnn.BF16 if dtype == "bf16" else mpcnn.F32)
    plan = net.plan_describe(B, H, W, False)
    assert (AT_END in plan or not at_end) and AT_END not in net.plan_describe(B, H, W, True), plan
    if seen is not None:
        line = [l for l in plan.splitlines() if "forward:" in l][-1]
        seen.add(line.split("waves ")[1].split(" channels and")[0])
    rng = np.random.default_rng(H + W)
    if params is None:
        params, ci = [], 1
        side = patch
        for kind, m, k in layers:
            if kind == MP:
                side //= k
                continue
            f = k if kind == C else side
            side = side - k + 1 if kind == C else 1
            params.append(rng.uniform(-1, 1, m * ci * f * f + m) * 1.5 / np.sqrt(ci * f * f))
            ci = m
        params = np.concatenate(params)
    net.set_params(params.astype(np.float32))
    net.set_loss(loss)
    net.set_activation(squash)
    image = torch.from_numpy(rng.uniform(0, 1, (B, 1, H, W)).astype(np.float32)).cuda()
    labels = torch.from_numpy(rng.integers(-1, layers[-1][1] + 1, (B, H, W)).astype(np.int32)).cuda()
    pixw = torch.from_numpy(rng.uniform(0.5, 2, (B, H, W)).astype(np.float32)).cuda()
    probs = torch.full((B, layers[-1][1], H - patch + 1, W - patch + 1), -1.0, device="cuda")
    total = torch.zeros(1, dtype=torch.float64, device="cuda")
    net.seg_backward(image, labels, pixw=pixw, probs=probs, loss=total)
    want = probs.cpu().numpy()
    got = net.seg_forward(image, torch.full_like(probs, -1.0)).cpu().numpy()
    assert np.array_equal(got, want, equal_nan=True), (layers, np.abs(got - want).max())
    # mirrored borders: the image mirrored by hand
    same = net.seg_forward_same(image).cpu().numpy()
    c = (patch - 1) // 2
    assert np.array_equal(same[:, :, c:c + want.shape[2], c:c + want.shape[3]], want, equal_nan=True)
    wide = np.pad(image.cpu().numpy(), ((0, 0), (0, 0), (c, patch - 1 - c), (c, patch - 1 - c)), mode="symmetric")
    assert np.array_equal(same, net.seg_forward(torch.from_numpy(wide).cuda()).cpu().numpy(), equal_nan=True)
    only = net.seg_loss(image, labels, pixw=pixw)
    net.close()
    # a pixel's squared error is formed in fp32 (2^-24 of it, where one kernel fuses a multiply-add that the other does not), the sum in fp64
    if np.isfinite(total.item()):
        assert abs(only - total.item()) <= 2.0 ** -23 * abs(total.item())
    return want


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_bits_of_the_training_pass(dtype):
    seen = set()
    for hidden, classes, below, k, sizes in (
            (100, 2, 64, 3, ((50, 55), (200, 171))), (200, 3, 128, 2, ((75, 60), (300, 410))), (128, 2, 32, 2, ((61, 40),)), (160, 3, 32, 4, ((90, 71),)), (164, 2, 20, 2, ((57, 49),)), (132, 2, 20, 2, ((70, 36),)), (256, 4, 48, 2, ((50, 55), (500, 470))),
            (68, 2, 16, 3, ((39, 41),)), (100, 2, 64, 2, ((900, 830),))):
        if below == 16 and dtype == "bf16":
            continue                                   # (no instance of such narrow blocks)
        layers = ((C, 8, 3), (MP, 0, 2), (C, below, 3), (FC, hidden, 0), (FC, classes, 0))
        patch = 2 * (k + 2) + 2                        # -> 2 (k + 2) -> k + 2 -> k
        for i, (h, w) in enumerate(sizes):
            check(layers, patch, 1 + i, patch + h, patch + w, dtype, ("mcce", "mse")[i % 2], ("tanh", "logistic")[hidden % 3 % 2], seen)
    text = (Path(mpcnn.__file__).parent / "csrc" / "launchers.hpp").read_text()
    text = text[text.index("#define MPCNN_HEAD%d(" % (3 if dtype == "f32" else 1)):].split("\n")[0]
    want = {"%s x %s of %s x %s tiles, %s" % (f[1:] + f[:1]) for f in re.findall(r"X\((\d+), (\d+), (\d+), (\d+), (\d+)\)", text)}
    assert want and seen == want, (sorted(want - seen), sorted(seen - want))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,classes,below,k,height,width", [
    (100, 2, 64, 3, 40, 47), (200, 3, 128, 2, 36, 70), (160, 3, 32, 4, 50, 55), (132, 2, 20, 2, 44, 39), (256, 4, 48, 2, 45, 38)])
def test_bits_of_the_training_pass_on_few_positions(hidden, classes, below, k, height, width, dtype):
    """Maps of few tiles: the class layer at the end, or in a launch of its own where that is faster."""
    layers = ((C, 8, 3), (MP, 0, 2), (C, below, 3), (FC, hidden, 0), (FC, classes, 0))
    patch = 2 * (k + 2) + 2
    check(layers, patch, 1, patch + height, patch + width, dtype, "mcce", ("tanh", "logistic")[hidden % 3 % 2], at_end=False)


@pytest.mark.parametrize("H,W", [(60, 51), (140, 131)])
@pytest.mark.parametrize("hidden", [100, 200])
def test_sums_that_are_not_finite(hidden, H, W):
    """Infinite weights: outputs as they are without parts, repaired in memory on their way to the classes; a NaN pixel: its patches alone."""
    layers = ((C, 16, 3), (C, 64, 3), (FC, hidden, 0), (FC, 2, 0))
    patch, at_end = 8, H > 100
    rng = np.random.default_rng(hidden)
    n = [16 * 9 + 16, 64 * 16 * 9 + 64, hidden * 64 * 16 + hidden, 2 * hidden + 2]
    params = np.concatenate([rng.uniform(-1, 1, m) * s for m, s in zip(n, (0.5, 0.1, 0.05, 0.2))])
    params[n[0] + n[1] + 5] = np.inf
    params[n[0] + n[1] + 64 * 16 * (hidden - 1) + 7] = -np.inf
    want = check(layers, patch, 1, H, W, "f32", "mcce", "tanh", params=params, at_end=at_end)
    assert np.isfinite(want).all()
    params[3] = np.nan
    check(layers, patch, 1, H, W, "f32", "mcce", "tanh", params=params, at_end=at_end)


@pytest.mark.parametrize("H,W", [(30, 41), (80, 71)])
@pytest.mark.parametrize("hidden", [100, 200])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinite_pixels(hidden, dtype, H, W):
    """A hidden layer on the image itself: infinite inputs reach units that exist, and none of the channels that only fill the tiles."""
    net = mpcnn.Net(((FC, hidden, 0), (FC, 2, 0)), 20, 3, mpcnn.BF16 if dtype == "bf16" else mpcnn.F32)
    assert AT_END in net.plan_describe(1, H, W, False) or H < 50
    rng = np.random.default_rng(hidden)
    net.set_params(rng.uniform(-0.2, 0.2, net.param_count).astype(np.float32))
    image = rng.uniform(0, 1, (1, 20, H, W)).astype(np.float32)
    image[0, 3, 7, 9], image[0, 5, 20, 30] = np.inf, -np.inf
    image = torch.from_numpy(image).cuda()
    probs = torch.empty((1, 2, H - 2, W - 2), device="cuda")
    net.seg_backward(image, torch.zeros((1, H, W), dtype=torch.int32, device="cuda"), probs=probs)
    want = probs.cpu().numpy()
    assert np.isfinite(want).all()
    assert np.array_equal(net.seg_forward(image, torch.full_like(probs, -1.0)).cpu().numpy(), want)
    net.close()


@pytest.mark.parametrize("below,k,hidden,size", [(64, 2, 200, 300), (128, 2, 200, 310), (100, 3, 132, 300), (100, 3, 164, 300), (128, 2, 256, 400)])
def test_all_channels_in_one_workgroup(below, k, hidden, size):
    """bf16 storage, training: 161 .. 256 channels in one group of workgroups against two groups of four tiles (by a tiling hint), bit for bit."""
    layers = ((C, 8, 3), (MP, 0, 2), (C, below, 3), (FC, hidden, 0), (FC, 3, 0))
    patch = 2 * (k + 2) + 2
    H, W = patch + size, patch + size + 13
    rng = np.random.default_rng(below + hidden)
    n = [8 * 9 + 8, below * 8 * 9 + below, hidden * below * k * k + hidden, 3 * hidden + 3]
    params = np.concatenate([rng.uniform(-1, 1, m) * s for m, s in zip(n, (0.5, 0.2, 0.08, 0.2))]).astype(np.float32)
    image = torch.from_numpy(rng.uniform(0, 1, (1, 1, H, W)).astype(np.float32)).cuda()
    labels = torch.from_numpy(rng.integers(0, 3, (1, H, W)).astype(np.int32)).cuda()
    out = []
    for hint in ((0, 0), (4, 4)):
        net = mpcnn.Net(layers, 1, patch, mpcnn.BF16)
        net.set_conv_tiling(*hint)
        line = [l for l in net.plan_describe(1, H, W, True).splitlines() if "forward:" in l][-1]
        assert ("8 channel tiles x 1 groups" in line) == (hint == (0, 0) and hidden > 160), line
        net.set_params(params)
        probs = torch.empty((1, 3, H - patch + 1, W - patch + 1), device="cuda")
        net.seg_backward(image, labels, probs=probs)
        out.append((probs.cpu().numpy(), net.get_grads()))
        net.close()
    assert np.isfinite(out[0][1]).all() and np.any(out[0][1])
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,classes", [(4, 2), (24, 3), (60, 4), (64, 2), (68, 3), (100, 4), (128, 2), (132, 3), (136, 4), (160, 2), (180, 4), (192, 3), (196, 2), (200, 4), (256, 3)])
def test_class_layer_of_its_own(hidden, classes, dtype):
    """Training: one to four quads of channels per lane, whole and not, every number of classes; against the oracle."""
    layers = ((C, 8, 3), (MP, 0, 2), (FC, hidden, 0), (FC, classes, 0))
    full_parity(wl.Workload("class_%d_%d_%s" % (hidden, classes, dtype), layers, 6, 1, classes, 2, 31, 24, 0.3, "ellipses", dtype=dtype,
                            seed_image=1611 + hidden, seed_label=2611, seed_param=3611), with_pixw=True, ignore_some=True,
                loss_fn="mse" if hidden % 16 else "mcce")
