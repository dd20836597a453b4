"""Setting and reading parameters on both sides of the size up to which the host permutes a vector, and of the number of launches that carry it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1302_1690_amd import mpcnn, workloads as wl

pytestmark = pytest.mark.gpu
C, MP, FC = wl.C, wl.MP, wl.FC


@pytest.mark.parametrize("maps,fc,count", [(1, 1, 19), (5, 39, 949), (10, 20, 962), (7, 63, 2025), (7, 64, 2056), (16, 100, 6862), (40, 300, 49302)])
def test_round_trip(maps, fc, count):
    # patch 6 -> (C 3x3) 4 -> (MP2) 2 -> FC over 2x2
    net = mpcnn.Net(((C, maps, 3), (MP, 0, 2), (FC, fc, 0), (FC, 2, 0)), 1, 6)
    p = np.random.default_rng(maps).standard_normal(count).astype(np.float32)
    net.set_params(p)                       # (refuses any other count)
    assert np.array_equal(net.get_params(), p)
