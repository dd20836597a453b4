"""The image layer and the 2 x 2 pool behind it in one launch (forward passes that keep nothing, fp32 storage) against the training pass, which makes
two, bit for bit: filter sides, channels, rows per wave, ragged tiles, a pool that drops a row, mirrored borders, a NaN and ties."""
import numpy as np
import pytest
import torch

from paper_1302_1690_amd import mpcnn, workloads as wl

C, MP, FC = wl.C, wl.MP, wl.FC
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ch", [1, 3])
@pytest.mark.parametrize("k,maps,patch", [(3, 12, 10), (5, 33, 12), (7, 64, 15), (5, 10, 13)])
@pytest.mark.parametrize("batch,height,width", [(2, 3, 5), (1, 31, 63), (3, 150, 97), (1, 640, 500)])
def test_bits_of_two_launches(ch, k, maps, patch, batch, height, width):
    layers = ((C, maps, k), (MP, 0, 2), (FC, 12, 0), (FC, 2, 0))     # (5, 10, 13): a map of 9, whose last row and column no window covers
    H, W = patch + height, patch + width
    rng = np.random.default_rng(1000 * k + width)
    net = mpcnn.Net(layers, ch, patch)
    n = [maps * ch * k * k + maps]
    side = (patch - k + 1) // 2
    n += [12 * maps * side * side + 12, 26]
    net.set_params(np.concatenate([rng.uniform(-1, 1, m) * s for m, s in zip(n, (0.4, 0.1, 0.3))]).astype(np.float32))
    net.set_activation("logistic" if width == 97 else "tanh")
    image = rng.uniform(0, 1, (batch, ch, H, W)).astype(np.float32)
    image[0, 0, 2:9, 1:9] = 0.25                       # windows whose values are equal
    if height == 150:
        image[1, ch - 1, 60, 50] = np.nan
    image = torch.from_numpy(image).cuda()
    labels = torch.zeros((batch, H, W), dtype=torch.int32, device="cuda")
    probs = torch.empty((batch, 2, height + 1, width + 1), device="cuda")
    net.seg_backward(image, labels, probs=probs)
    want = probs.cpu().numpy()
    assert np.isfinite(want).all() == (height != 150)
    got = net.seg_forward(image, torch.full_like(probs, -1.0)).cpu().numpy()
    assert np.array_equal(got, want, equal_nan=True)
    # borders: the same image mirrored by hand
    same = net.seg_forward_same(image).cpu().numpy()
    c = (patch - 1) // 2
    wide = np.pad(image.cpu().numpy(), ((0, 0), (0, 0), (c, patch - 1 - c), (c, patch - 1 - c)), mode="symmetric")
    by_hand = net.seg_forward(torch.from_numpy(wide).cuda()).cpu().numpy()
    assert np.array_equal(same, by_hand, equal_nan=True)
    net.close()
