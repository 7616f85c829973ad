"""A depthwise convolution and the 1x1 convolution behind it in one launch: the bits of the two launches, in the output
and in the depthwise tensor.  The separate launches are compared with the oracle layer by layer elsewhere."""

import pytest
import torch

from paper_2109_01611_amd import gpulet, lowering, workloads
from paper_2109_01611_amd.workloads import Model, _conv, _dwconv

from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _pair(C, H, W, K, relu=True, stride=1):
    return Model("pair", (C, H, W), "normal", [
        _dwconv("d", "x", "t", C, 3, stride, 1, relu),
        _conv("c", "t", "y", C, K, 1, 1, 0, relu),
    ], "y")


# C, H, W, K, batch, percent: odd maps, maps smaller than a block, tiles that span images, a ragged last tile, several
# workgroups per tile, both widths of filter tiles and heights of pixel tiles of the deep kernel
CASES = [
    (32, 21, 18, 64, 19, 25), (32, 1, 1, 64, 1024, 25), (32, 9, 50, 128, 8, 25), (32, 40, 37, 64, 30, 25),
    (128, 9, 11, 128, 4, 100), (128, 10, 10, 384, 3, 100), (128, 30, 31, 128, 8, 20),
    (192, 7, 5, 128, 2, 100), (192, 28, 28, 128, 8, 60), (256, 9, 9, 256, 3, 100), (256, 38, 38, 256, 8, 100),
    (320, 5, 6, 384, 2, 100), (512, 19, 19, 512, 1, 60), (512, 19, 19, 512, 8, 100), (512, 3, 2, 256, 1, 100),
    (512, 10, 10, 1024, 16, 100), (256, 18, 19, 256, 6, 25),
]
# two launches: stride 2, other channel counts, more than one round of the deep kernel, filters no multiple of a tile, 32 channels
# on few workgroups
SEPARATE = [
    (32, 21, 18, 64, 3, 100, 1), (32, 1, 1, 64, 1, 100, 1), (32, 9, 50, 128, 2, 100, 1),
    (32, 21, 18, 64, 3, 100, 2), (64, 14, 9, 128, 3, 100, 1), (1024, 5, 5, 1024, 1, 100, 1), (512, 19, 19, 512, 32, 100, 1),
    (128, 9, 11, 72, 1, 100, 1), (32, 9, 11, 96, 1, 100, 1), (40, 9, 11, 64, 1, 100, 1), (128, 75, 75, 128, 16, 20, 1),
]


def _both_ways(model, batch, pct, fused_launches, x=None, bias=True):
    dm = lowering.DeviceModel(model, workloads.parameters(model, 5), DEV)
    if not bias:
        for layer in dm.layers:
            layer.b = None
    with gpulet.Partition(0, pct, 0) as p:
        xd = dm.input_to_device(workloads.batch_input(model, batch, 5) if x is None else x)
        seen = []
        for fused in (False, True):
            gpulet.set_conv_pool_fusion(fused)
            try:
                dm.workspace(batch)[0].fill_(255)
                before = p.kernel_launches()
                y, _ = dm.run(p, xd)
                assert p.kernel_launches() - before == (fused_launches if fused else 2)
            finally:
                gpulet.set_conv_pool_fusion(True)
            seen.append((y.clone(), dm.read_tensor("t", batch)))
    for a, b in zip(*seen):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(nan=0.0), b.nan_to_num(nan=0.0))
    return seen[1]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_pair_in_one_launch_is_the_two_launches(case):
    C, H, W, K, batch, pct = case
    for relu in (True, False):
        _both_ways(_pair(C, H, W, K, relu), batch, pct, 1)


# both kernels, both widths of filter tiles and heights of pixel tiles
EDGES = [(32, 40, 37, 64, 30, 25), (128, 9, 11, 128, 8, 100), (256, 9, 9, 256, 6, 100), (256, 38, 38, 256, 8, 100)]


@pytest.mark.parametrize("case", EDGES, ids=lambda c: "x".join(map(str, c)))
def test_no_bias(case):
    C, H, W, K, batch, pct = case
    _both_ways(_pair(C, H, W, K, False), batch, pct, 1, bias=False)


@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("case", EDGES, ids=lambda c: "x".join(map(str, c)))
def test_infinities_and_nan(case, relu):
    # in the corners and the middle of some images; those between them have to stay finite
    C, H, W, K, batch, pct = case
    model = _pair(C, H, W, K, relu)
    x = workloads.batch_input(model, batch, 5)
    x[0, 1, 0, 0] = float("inf")
    x[1, C - 1, H - 1, W - 1] = -float("inf")
    x[2, 0, H // 2, W // 2] = float("nan")
    x[3] = -3.3895e38
    for t in _both_ways(model, batch, pct, 1, x=x):
        assert t[4:].isfinite().all()
        assert t[:3].isfinite().float().mean() > 0.5   # pixels whose window does not touch them


@pytest.mark.parametrize("case", SEPARATE, ids=lambda c: "x".join(map(str, c)))
def test_pairs_that_stay_two_launches(case):
    C, H, W, K, batch, pct, stride = case
    _both_ways(_pair(C, H, W, K, True, stride), batch, pct, 2)


def test_a_depth_split_keeps_its_sums():
    gpulet.set_conv_split_k(8)
    try:
        _both_ways(_pair(512, 10, 10, 512), 1, 100, 2)
    finally:
        gpulet.set_conv_split_k(1)


@pytest.mark.parametrize("reuse", [True, False])
def test_whole_model_with_and_without_shared_launches(reuse):
    model = workloads.ssd_mobilenet()
    params = workloads.parameters(model, 6)
    dm = lowering.DeviceModel(model, params, DEV, reuse=reuse)
    with gpulet.Partition(0, 80, 0) as p:
        xd = dm.input_to_device(workloads.batch_input(model, 3, 6))
        out = []
        for fused in (False, True):
            gpulet.set_conv_pool_fusion(fused)
            try:
                dm.workspace(3)[0].fill_(255)   # what a launch leaves out stays NaN
                before = p.kernel_launches()
                y, _ = dm.run(p, xd)
                n = p.kernel_launches() - before
            finally:
                gpulet.set_conv_pool_fusion(True)
            out.append((n, [y.clone()] + ([] if reuse else [dm.read_tensor(t, 3) for t in dm.tensor_buf if dm.tensor_buf[t] != 1])))
    assert out[1][0] < out[0][0]
    assert all(torch.equal(a, b) for a, b in zip(out[0][1], out[1][1]))
