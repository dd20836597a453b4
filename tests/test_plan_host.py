"""Which kernels the planner gives to convolutions (no GPU): large filters and wide layers stay on the matrix cores; the weight gradient's
kernel by the size of its work."""
import pytest

from paper_1302_1690_amd import mpcnn, workloads as wl

C, MP, FC = wl.C, wl.MP, wl.FC


def conv_lines(layers, patch, size, dtype, layer):
    net = mpcnn.Net(layers, 1, patch, dtype)
    plan = net.plan_describe(1, size, size, True)
    net.close()
    own = plan[plan.index("layer %d:" % layer):plan.index("layer %d:" % (layer + 1))]
    return [line for line in own.splitlines() if "forward:" in line or "data gradient:" in line]


@pytest.mark.parametrize("dtype", [mpcnn.F32, mpcnn.BF16])
@pytest.mark.parametrize("channels", [8, 12, 16, 32, 64])
def test_large_filters_are_on_the_matrix_cores(channels, dtype):
    """Up to 48 x 48; those whose halo holds fewer positions than a workgroup's tile in blocks of fewer rows."""
    for k in (2, 7, 8, 20, 25, 26, 33, 43, 48):
        lines = conv_lines(((C, channels, 3), (C, 32, k), (MP, 0, 2), (FC, 16, 0), (FC, 2, 0)), k + 6, 2 * k + 90, dtype, 1)
        assert len(lines) == 2
        for line in lines:
            assert "plain" not in line, (k, line)
            rows = int(line.split(" filter rows")[0].split()[-1])
            assert rows == k if k < 8 else 1 <= rows <= k, (k, line)


@pytest.mark.parametrize("dtype", [mpcnn.F32, mpcnn.BF16])
@pytest.mark.parametrize("k,cin,cout", [(5, 4000, 4000), (5, 4500, 64), (9, 2048, 2400), (1, 22000, 8)])
def test_wide_layers_are_on_the_matrix_cores(k, cin, cout, dtype):
    """Layers of up to 2 GiB of parameters (their packs are larger: rounded up, and three parts of two bytes per number with fp32 storage)."""
    for line in conv_lines(((C, cin, 3), (C, cout, k), (FC, 16, 0), (FC, 2, 0)), k + 4, k + 20, dtype, 1):
        assert "plain" not in line, line


@pytest.mark.parametrize("size,parts", [(10, False), (40, False), (71, True), (300, True)])
def test_weight_gradient_kernel_by_its_work(size, parts):
    """16 -> 40 channels, 3 x 3: from 4e7 operations on in three parts per number."""
    net = mpcnn.Net(((C, 16, 3), (C, 40, 3), (FC, 24, 0), (FC, 2, 0)), 1, 8)
    plan = net.plan_describe(1, size, size, True)
    net.close()
    own = plan[plan.index("layer 1:"):plan.index("layer 2:")]
    assert ("weight gradient: bf16 MFMA, three parts" in own) == parts, own
    assert ("weight gradient: fp32 MFMA" in own) != parts, own


@pytest.mark.parametrize("classes", [2, 4, 5])
def test_two_parts_where_a_launch_may_take_them(classes):
    """Five classes are not the fused class layer's, so nobody notes how large the deltas above the hidden layer are: three parts there, planned and said; two in the layer below, whose deltas
    a data gradient has written."""
    net = mpcnn.Net(((C, 64, 3), (C, 64, 3), (FC, 128, 0), (FC, classes, 0)), 1, 7)
    plan = net.plan_describe(1, 210, 200, True)
    net.close()
    said = {}
    for layer in (1, 2):
        own = plan[plan.index("layer %d:" % layer):plan.index("layer %d:" % (layer + 1))]
        for line in own.splitlines():
            if "MFMA" in line:
                said[layer, line.split(":")[0].strip()] = "or two of fp16" in line
    known = classes <= 4
    assert said[1, "forward"] and said[1, "data gradient"] and said[2, "forward"], plan
    assert said[2, "data gradient"] == known and said[2, "weight gradient"] == known, plan


@pytest.mark.parametrize("training", [True, False])
@pytest.mark.parametrize("maps,k", [(1, 3), (3, 5), (3, 7)])
def test_narrow_layers_are_on_the_matrix_cores(maps, k, training):
    """A second convolution on one or three maps is the fp32 instruction's, as the image layer is; behind a pool (spacing 2) it is not."""
    def forward(layers, patch, layer):
        net = mpcnn.Net(layers, 3, patch)
        plan = net.plan_describe(1, 512, 512, training)
        net.close()
        own = plan[plan.index("layer %d:" % layer):plan.index("layer %d:" % (layer + 1))]
        return [line for line in own.splitlines() if "forward:" in line][0]

    rest = ((MP, 0, 2), (FC, 20, 0), (FC, 2, 0))
    assert "on the fp32 MFMA" in forward(((C, maps, 3), (C, 64, k)) + rest, k + 5, 1)
    assert "plain kernel" in forward(((C, maps, 3), (MP, 0, 2), (C, 64, k)) + rest, 2 * k + 4, 2)


def test_nets_in_one_launch_are_those_it_is_faster_for():
    """Nothing for the convolutions' matrix instruction and eight channels at most; of these, nets of three layers and more, without convolutions of four or
    eight maps, of 150 filter taps and 64 on a single map, whose squares hold 14 x 14 pixels at two thirds of halo: at every size, in every call, and with a tiling,
    which promises the same bits."""
    def small(layers, patch, size, training, ch=1, hint=(0, 0)):
        net = mpcnn.Net(layers, ch, patch)
        net.set_conv_tiling(*hint)
        plan = net.plan_describe(1, size, size, training)
        net.close()
        return "whole net in one launch" in plan

    tiny = wl.CONFIGS[0]
    refused = [(((C, 8, 5), (MP, 0, 2), (FC, 7, 0), (FC, 2, 0)), 14), (((C, 8, 3), (MP, 0, 2), (FC, 2, 0), (FC, 3, 0)), 14),
               (((C, 4, 3), (MP, 0, 2), (FC, 4, 0), (FC, 2, 0)), 10), (((FC, 3, 0),), 4), (((FC, 8, 0), (FC, 2, 0)), 6),
               (((C, 7, 7), (FC, 5, 0), (FC, 2, 0)), 7), (((C, 1, 5), (MP, 0, 3), (FC, 6, 0), (FC, 2, 0)), 22), (((C, 5, 3), (MP, 0, 3), (FC, 4, 0), (FC, 2, 0)), 14),
               (((MP, 0, 3), (C, 5, 2), (MP, 0, 2), (FC, 4, 0), (FC, 2, 0)), 17), (((C, 9, 3), (FC, 3, 0), (FC, 2, 0)), 4),
               (((C, 8, 3), (C, 8, 3), (FC, 2, 0)), 6), (((C, 7, 9), (C, 7, 9), (FC, 2, 0)), 17)]
    for size in (40, 64, 301, 1024, 2048):
        for training in (False, True):
            assert small(tiny.layers, tiny.patch, size, training) and small(tiny.layers, tiny.patch, size, training, hint=(4, 1))
            assert small(((C, 7, 2), (C, 3, 5), (FC, 5, 0), (FC, 2, 0)), 6, size, training, 3)
            for layers, patch in refused:
                assert not small(layers, patch, size, training, 2 if patch == 17 else 1), layers


@pytest.mark.parametrize("channels,k,maps,rows_of", [
    (1, 3, 16, {80: 1, 256: 1, 600: 2, 1400: 2}), (1, 7, 64, {150: 1, 256: 2, 512: 2, 1024: 2}), (3, 5, 64, {112: 1, 360: 2, 1024: 2}),
    (3, 7, 32, {256: 1, 300: 2, 512: 2, 600: 2}), (3, 7, 128, {112: 2, 256: 2, 420: 2, 1024: 4})])
def test_rows_per_wave_of_the_image_layer_with_the_pool(channels, k, maps, rows_of):
    """The one that was measured to be the fastest, at sizes where the others take 2 to 20 % more of a forward pass."""
    net = mpcnn.Net(((C, maps, k), (MP, 0, 2), (FC, 12, 0), (FC, 2, 0)), channels, k + 5)
    for size, rows in rows_of.items():
        assert "same launch, %d rows per wave" % rows in net.plan_describe(1, size, size + 9, False), size
    net.close()


@pytest.mark.parametrize("dtype,below,k,units,at_end", [
    (mpcnn.F32, 64, 3, 100, {50: True, 97: True, 300: True, 1000: True}), (mpcnn.F32, 128, 2, 200, {40: False, 97: True, 600: True}),
    (mpcnn.F32, 64, 5, 200, {40: False, 60: False, 200: True, 600: True}), (mpcnn.F32, 32, 3, 132, {40: False, 97: True, 300: False, 600: False, 1000: False}),
    (mpcnn.F32, 32, 3, 160, {40: False, 430: False}), (mpcnn.F32, 64, 3, 132, {300: False}), (mpcnn.F32, 64, 3, 160, {97: True, 300: True, 1000: True}),
    (mpcnn.BF16, 64, 5, 68, {40: False, 60: False, 300: True}), (mpcnn.BF16, 128, 2, 68, {40: False, 60: False, 200: True}),
    (mpcnn.BF16, 32, 3, 132, {97: True, 600: True}), (mpcnn.BF16, 64, 3, 200, {40: True, 300: True}), (mpcnn.BF16, 128, 2, 200, {97: True, 300: True, 1000: True})])
def test_class_layer_at_the_end_where_it_is_faster(dtype, below, k, units, at_end):
    """Not on maps of few tiles behind long sums, nor where five tiles leave the eight waves of fp32 storage half empty."""
    net = mpcnn.Net(((C, 8, 3), (MP, 0, 2), (C, below, 3), (FC, units, 0), (FC, 2, 0)), 1, 2 * (k + 2) + 2, dtype)
    for size, want in at_end.items():
        assert ("class layer: at the end of the layer below" in net.plan_describe(1, size, size + 7, False)) == want, size
    net.close()


@pytest.mark.parametrize("below,k", [(64, 3), (128, 2)])
@pytest.mark.parametrize("units,groups", [(132, 2), (160, 2), (164, 1), (200, 1), (256, 1)])
def test_wide_layers_in_one_group_where_its_waves_are_busy(below, k, units, groups):
    """bf16 storage, large maps: two groups of four tiles where one of eight would have no more than five."""
    forward = conv_lines(((C, 8, 3), (MP, 0, 2), (C, below, 3), (FC, units, 0), (FC, 2, 0)), 2 * (k + 2) + 2, 1400, mpcnn.BF16, 3)[0]
    assert "x %d groups" % groups in forward, forward


@pytest.mark.parametrize("dtype", [mpcnn.F32, mpcnn.BF16])
def test_class_layer_at_the_end_of_few_positions_of_many_residue_classes(dtype):
    """Behind four pools even a map of 4 x 21 positions has a workgroup for every compute unit."""
    net = mpcnn.Net(((C, 32, 7), (MP, 0, 2), (C, 64, 5), (MP, 0, 2), (C, 64, 5), (MP, 0, 2), (C, 128, 3), (MP, 0, 2), (FC, 200, 0), (FC, 2, 0)), 1, 78, dtype)
    assert "class layer: at the end of the layer below" in net.plan_describe(1, 81, 98, False)
    net.close()


def test_pool_behind_the_image_layer_is_a_launch_where_that_is_faster():
    """7 x 7 filters on three channels, 128 maps: what a tile computes twice is dearer than the pool's launch where workgroups would wait for a second round."""
    net = mpcnn.Net(((C, 128, 7), (MP, 0, 2), (FC, 12, 0), (FC, 2, 0)), 3, 12)
    for height, width, fused in ((64, 64, True), (200, 209, False), (256, 256, False), (256, 265, True), (512, 512, True), (1024, 1024, True)):
        assert ("the pool behind it in the same launch" in net.plan_describe(1, height, width, False)) == fused, (height, width)
    net.close()
