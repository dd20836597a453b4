"""Weight gradient of the image layer with bf16 storage (csrc/kernels_l0_wgrad.hpp): filter sides 3, 5, 7, one and three input
channels, map counts of one and two slices that are and are not a multiple of 8, images that end inside a tile in both
directions, more tiles than workgroups; full oracle."""
import pytest

torch = pytest.importorskip("torch")

from paper_1302_1690_amd import mpcnn, workloads as wl
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
C, MP, FC = wl.C, wl.MP, wl.FC

CASES = [  # (k, channels, maps, height, width, batch)
    (3, 1, 8, 41, 37, 2), (5, 1, 48, 45, 70, 1), (7, 1, 16, 52, 66, 1), (3, 3, 40, 38, 35, 1), (5, 3, 32, 45, 71, 2),
    (7, 3, 24, 49, 40, 1), (5, 3, 8, 10, 10, 1), (5, 3, 12, 45, 37, 1), (3, 1, 8, 330, 450, 2),
]


@pytest.mark.parametrize("k,ci,maps,height,width,batch", CASES)
def test_weight_gradient_with_bf16_storage(k, ci, maps, height, width, batch):
    # patch: k + 5 -> 6 -> (C 3x3) 4 -> (MP2) 2 -> FC over 2x2 (no pool behind the image layer: with one, small images go to the fused kernel)
    layers = ((C, maps, k), (C, 8, 3), (MP, 0, 2), (FC, 6, 0), (FC, 2, 0))
    plan = mpcnn.Net(layers, ci, k + 5, 1).plan_describe(batch, height, width, True)
    assert "image-layer kernel on the %s MFMA, " % ("bf16" if maps % 8 == 0 else "fp32") in plan
    full_parity(wl.Workload("image_layer_bf16_k%d_c%d_m%d" % (k, ci, maps), layers, k + 5, ci, 2, batch, height, width, 0.2,
                            "ellipses", dtype="bf16", seed_image=1401, seed_label=2401, seed_param=3401), with_pixw=True)


@pytest.mark.parametrize("maps,k", [(1, 5), (3, 3), (3, 7)])
def test_a_later_layer_as_narrow(maps, k):
    """fp32 storage: a second convolution on one or three maps takes the image layer's kernel."""
    layers = ((C, maps, 3), (C, 12, k), (MP, 0, 2), (FC, 6, 0), (FC, 2, 0))
    plan = mpcnn.Net(layers, 3, k + 5).plan_describe(2, 60, 77, True)
    assert "on the fp32 MFMA" in plan[plan.index("layer 1:"):plan.index("layer 2:")].split("gradient")[0]
    full_parity(wl.Workload("narrow_k%d_m%d" % (k, maps), layers, k + 5, 3, 2, 2, 60, 77, 0.3, "ellipses",
                            seed_image=1402, seed_label=2402, seed_param=3402), with_pixw=True)
