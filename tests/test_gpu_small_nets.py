"""Nets of few maps and parameters, whose whole pass is one launch (squares of output pixels through every layer, forward and back): against the
oracle, at sizes of one square and less, a ragged last one and several per workgroup, over the filters, windows, spacings and channel counts the
kernel takes; and against the layer-by-layer kernels, which a twin with more hidden units, all of them zeros, is left to."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_1302_1690_amd import mpcnn, workloads as wl
from test_gpu_parity import full_parity, run_gpu

C, MP, FC = wl.C, wl.MP, wl.FC
pytestmark = pytest.mark.gpu

NETS = [   # name, layers, patch, image channels
    ("tiny", wl.CONFIGS[0].layers, wl.CONFIGS[0].patch, 1),
    ("fc_only", ((FC, 3, 0), (FC, 4, 0), (FC, 2, 0)), 4, 1),
    ("pool_first_dropping", ((MP, 0, 3), (C, 5, 2), (MP, 0, 2), (FC, 4, 0), (FC, 2, 0)), 11, 2),   # 11 -> 3 (2 left over) -> 2 -> 1
    ("seven_maps_three_channels", ((C, 7, 3), (MP, 0, 2), (C, 7, 2), (FC, 6, 0), (FC, 5, 0)), 6, 3),
    ("one_map_each", ((C, 1, 1), (C, 1, 4), (MP, 0, 4), (FC, 1, 0), (FC, 8, 0)), 7, 1),
    ("more_parameters_than_threads", ((C, 7, 2), (C, 3, 5), (FC, 5, 0), (FC, 2, 0)), 6, 3),
]
LAYER_BY_LAYER = [   # as few maps, but slower in one launch where images are large
    ("one_layer", ((FC, 3, 0),), 4, 1),
    ("halo", ((MP, 0, 3), (C, 5, 2), (MP, 0, 2), (FC, 4, 0), (FC, 2, 0)), 17, 2),                  # 17 -> 5 (2 left over) -> 4 -> 2
    ("squares_of_12", ((C, 7, 3), (MP, 0, 2), (C, 7, 3), (FC, 6, 0), (FC, 5, 0)), 8, 3),
    ("taps", ((C, 6, 7), (C, 6, 4), (FC, 5, 0), (FC, 2, 0)), 12, 3),
    ("taps_on_one_map", ((C, 1, 5), (MP, 0, 3), (FC, 6, 0), (FC, 2, 0)), 22, 1),
    ("eight_maps", ((C, 8, 5), (MP, 0, 2), (FC, 7, 0), (FC, 2, 0)), 14, 1),
]


def small(layers, patch, ch, B, H, W, training=True):
    net = mpcnn.Net(layers, ch, patch)
    plan = net.plan_describe(B, H, W, training)
    net.close()
    return "whole net in one launch" in plan


@pytest.mark.parametrize("name,layers,patch,ch", NETS + LAYER_BY_LAYER, ids=[n[0] for n in NETS + LAYER_BY_LAYER])
@pytest.mark.parametrize("over", [(0, 0), (2, 5), (26, 17)])
def test_against_the_oracle(name, layers, patch, ch, over):
    assert small(layers, patch, ch, 2, patch + over[0], patch + over[1]) == any(name == n[0] for n in NETS)
    full_parity(wl.Workload("small_" + name, layers, patch, ch, layers[-1][1], 2, patch + over[0], patch + over[1], 0.4, "ellipses" if ch == 3 else "bernoulli",
                            seed_image=1211, seed_label=2211, seed_param=3211), with_pixw=True, ignore_some=over[0] > 20)


def net_or_twin(cfg, params, hidden):
    """cfg's net, or its twin that is run layer by layer: 12 hidden units instead of 8, four of them without weights into them or out of them.
    And which of its parameters are cfg's."""
    net = mpcnn.Net(cfg.layers[:-2] + ((FC, hidden, 0), cfg.layers[-1]), cfg.in_channels, cfg.patch)
    own = np.ones(net.param_count, dtype=bool)
    if hidden == 12:
        n_in = 3 * 3 * 3                               # W[o][c][u][v], b[o] of the hidden layer, then W[o][unit], b[o]
        at = net.param_count - (12 * n_in + 12) - (2 * 12 + 2)
        own[at + 8 * n_in:at + 12 * n_in] = False
        own[at + 12 * n_in + 8:at + 12 * n_in + 12] = False
        for o in range(2):
            own[net.param_count - 26 + 12 * o + 8:net.param_count - 26 + 12 * o + 12] = False
    wide = np.zeros(net.param_count, dtype=np.float32)
    wide[own] = params
    net.set_params(wide)
    return net, own


@pytest.mark.parametrize("loss,squash", [("mcce", "tanh"), ("mse", "logistic")])
@pytest.mark.parametrize("batch,height,width", [(1, 150, 133), (3, 300, 222)])
def test_against_the_layers_one_by_one(batch, height, width, loss, squash):
    """Several squares per workgroup at the larger size.  Both paths add the same products in fp32, in other orders: a few 1e-7 of an output; gradients
    sum 1e5 such pixels, and a window whose best two are that close may pass its delta on to either (1e-4 of a tensor's largest, as against the oracle)."""
    cfg = replace(wl.crop(wl.CONFIGS[0], batch, height, width), name="small_large")
    img, lab = wl.make_inputs(cfg)
    params = wl.make_params(cfg)
    d_img, d_lab = torch.from_numpy(img).cuda(), torch.from_numpy(lab).cuda()
    pixw = torch.rand(d_lab.shape, device="cuda") + 0.5
    out = []
    for hidden in (8, 12):
        net, own = net_or_twin(cfg, params, hidden)
        assert ("whole net" in net.plan_describe(batch, height, width, True)) == (hidden == 8)
        net.set_loss(loss)
        net.set_activation(squash)
        probs = torch.empty((batch, cfg.n_classes, cfg.out_h, cfg.out_w), device="cuda")
        total = torch.zeros(1, dtype=torch.float64, device="cuda")
        net.seg_backward(d_img, d_lab, pixw=pixw, probs=probs, loss=total)
        grads = net.get_grads()[own]
        same = net.seg_forward_same(d_img).cpu().numpy()
        only = net.seg_forward(d_img).cpu().numpy()
        p = probs.cpu().numpy()
        c = (cfg.patch - 1) // 2
        assert np.array_equal(only, p) and np.array_equal(same[:, :, c:c + cfg.out_h, c:c + cfg.out_w], p)
        banded = torch.zeros(1, dtype=torch.float64, device="cuda")
        net.seg_backward_banded(d_img, d_lab, 37, pixw=pixw, probs=probs, loss=banded)
        assert np.array_equal(probs.cpu().numpy(), p)
        assert abs(banded.item() - total.item()) <= 1e-6 * abs(total.item())
        g2 = net.get_grads()[own]
        assert np.abs(g2 - grads).max() <= 1e-5 * np.abs(grads).max()
        out.append((p, same, total.item(), grads))
        net.close()
    (p0, s0, l0, g0), (p1, s1, l1, g1) = out
    assert np.abs(p0 - p1).max() <= 2e-6 and np.abs(s0 - s1).max() <= 2e-6
    assert abs(l0 - l1) <= 1e-6 * abs(l1)
    assert np.abs(g0 - g1).max() <= 1e-4 * np.abs(g1).max()


@pytest.mark.parametrize("hint", [(4, 1), (16, 4), (2, 0)])
def test_a_tiling_changes_nothing(hint):
    """mpcnn_set_conv_tiling promises the same sums in the same order."""
    cfg = replace(wl.crop(wl.CONFIGS[0], 2, 75, 90), name="small_hint")
    img, lab = wl.make_inputs(cfg)
    out = []
    for h in ((0, 0), hint):
        net, probs, loss, grads = run_gpu(cfg, img, lab, wl.make_params(cfg), tiling=h)
        out.append((probs, grads, loss))
        net.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]


def test_which_nets():
    """Nothing for the convolutions' matrix instruction, eight channels, 2048 parameters, a halo no dearer than the pixels; fp32."""
    tiny = wl.CONFIGS[0]
    assert small(tiny.layers, tiny.patch, 1, 1, 40, 40) and small(tiny.layers, tiny.patch, 1, 4, 900, 900, False)
    for layers, patch in ((((C, 9, 3), (FC, 2, 0)), 4), (((C, 8, 3), (C, 8, 3), (FC, 2, 0)), 6), (((C, 7, 9), (C, 7, 9), (FC, 2, 0)), 17)):
        assert not small(layers, patch, 1, 1, 60, 60), layers


def test_nan_stays_where_it_is():
    """A pixel that is not a number: outputs whose patches hold it are the oracle's (the pools pass over it in all places of a window but the first),
    all others are as they were; gradients are not numbers where the oracle's are not."""
    cfg = wl.crop(wl.CONFIGS[0], 1, 70, 61)
    img, lab = wl.make_inputs(cfg)
    params = wl.make_params(cfg)
    net, probs, _, _ = run_gpu(cfg, img, lab, params)
    img[0, 0, 33, 30] = np.nan
    _, bad, loss, grads = run_gpu(cfg, img, lab, params, net=net)
    net.close()
    hit = np.zeros((cfg.out_h, cfg.out_w), dtype=bool)
    hit[33 - cfg.patch + 1:34, 30 - cfg.patch + 1:31] = True
    assert np.array_equal(bad[:, :, ~hit], probs[:, :, ~hit])
    ref = oracle.run(cfg.layers, cfg.in_channels, cfg.patch, params.astype(np.float64), img.astype(np.float64), lab, want_grads=True)
    assert np.isnan(bad[:, :, hit]).any() and np.array_equal(np.isnan(bad), np.isnan(ref["probs"]))
    assert np.nanmax(np.abs(bad - ref["probs"])) <= 1e-6
    assert np.isnan(loss) == np.isnan(ref["loss"])
    assert np.isnan(grads).any() and np.array_equal(np.isnan(grads), np.isnan(ref["grads"]))
