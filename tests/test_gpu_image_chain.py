"""Small layers of a model in one launch (one workgroup per image): the bits of the launches they stand for, in
the output and in every tensor that separate launches leave in the workspace.  The separate launches are compared with
the oracle layer by layer elsewhere."""

import pytest
import torch

from paper_2109_01611_amd import gpulet, lowering, workloads
from paper_2109_01611_amd.workloads import Model, _conv, _fc, _maxpool

from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _mixed():
    # strides, paddings, odd maps, a 3x3 / stride 2 pool with padding, 64 channels under a filter larger than 1x1,
    # feature counts that are no multiple of 8, more layers than one launch takes
    return Model("mixed", (16, 13, 11), "normal", [
        _conv("a", "x", "ta", 16, 24, 3, 2, 1, True),
        _maxpool("b", "ta", "tb", 3, 2, 1),
        _conv("c", "tb", "tc", 24, 64, 1, 1, 0, False),
        _conv("d", "tc", "td", 64, 40, 2, 1, 1, True),
        _maxpool("e", "td", "te", 2, 1, 0),
        _conv("f", "te", "tf", 40, 8, 1, 1, 0, True),
        _fc("g", "tf", "tg", 8 * 4 * 3, 30, True),
        _fc("h", "tg", "th", 30, 80, True),
        _fc("i", "th", "ti", 80, 50, True),
        _fc("j", "ti", "y", 50, 20, False),
    ], "y")


def _ends_in_a_map():
    return Model("map", (8, 9, 20), "normal", [
        _conv("a", "x", "ta", 8, 16, 5, 1, 2, True),
        _conv("b", "ta", "tb", 16, 32, 3, 1, 1, False),
        _maxpool("c", "tb", "y", 2, 2, 0),
    ], "y")


def _long_row(W):
    # 8 x 32 x W / 2 features: from 8192 on the fully connected kernel adds in another order
    return Model("row%d" % W, (8, 64, W), "normal", [
        _maxpool("a", "x", "ta", 2, 2, 0),
        _fc("b", "ta", "tb", 8 * 32 * (W // 2), 4, True),
        _fc("c", "tb", "y", 4, 2, False),
    ], "y")


@pytest.mark.parametrize("reuse", [True, False])
@pytest.mark.parametrize("model,batch,pct,launches", [
    (workloads.lenet5(), 1, 100, 1), (workloads.lenet5(), 32, 20, 1), (workloads.lenet5(), 300, 60, 1),
    (_mixed(), 3, 40, 2), (_ends_in_a_map(), 2, 100, 1),
    (_long_row(62), 3, 100, 1), (_long_row(64), 3, 100, 3)], ids=lambda v: getattr(v, "name", str(v)))
def test_layers_of_one_launch_leave_what_separate_launches_leave(model, batch, pct, launches, reuse):
    _both_ways(model, batch, pct, launches, reuse, workloads.batch_input(model, batch, 3))


def _both_ways(model, batch, pct, launches, reuse, x, bias=True):
    params = workloads.parameters(model, 3)
    dm = lowering.DeviceModel(model, params, DEV, reuse=reuse)
    if not bias:
        for layer in dm.layers:
            layer.b = None
    with gpulet.Partition(0, pct, 0) as p:
        xd = dm.input_to_device(x)
        tensors = {}
        for fused in (False, True):
            gpulet.set_conv_pool_fusion(fused)
            try:
                before = p.kernel_launches()
                ws, _ = dm.workspace(batch)
                ws.fill_(255 if reuse else 0)
                y, _ = dm.run(p, xd)
                assert p.kernel_launches() - before == (launches if fused else dm.desc.n_layers)
            finally:
                gpulet.set_conv_pool_fusion(True)
            named = [] if reuse else [nd.dst for nd in model.nodes if nd.dst != model.out]
            tensors[fused] = [y.clone()] + [dm.read_tensor(t, batch) for t in named]
    for a, b in zip(*tensors.values()):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(nan=0.0), b.nan_to_num(nan=0.0))
    return tensors[True]


def _pools(n, W):
    names = ["x"] + ["t%d" % i for i in range(n - 1)] + ["y"]
    return Model("pools%dx%d" % (n, W), (8, 16, W), "normal", [_maxpool("p%d" % i, names[i], names[i + 1], 3, 1, 1) for i in range(n)],
                 "y")


def _only_fc():
    # starts with a fully connected layer, feature counts that are no multiple of 8 behind it
    return Model("fc", (72, 1, 1), "normal", [_fc("a", "x", "ta", 72, 42, True), _fc("b", "ta", "tb", 42, 28, False),
                                              _fc("c", "tb", "y", 28, 10, False)], "y")


@pytest.mark.parametrize("model,batch,launches,bias", [
    (_pools(7, 75), 3, 1, True),      # tensors, zeros and nothing else: 152,064 of 155,648 bytes of LDS
    (_pools(7, 76), 2, 2, True),      # eight tensors and the zeros would be 64 bytes too many
    (_pools(2, 9), 70, 1, True), (_only_fc(), 5, 1, True),
    (_only_fc(), 5, 1, False), (_ends_in_a_map(), 2, 1, False), (workloads.lenet5(), 3, 1, False), (_mixed(), 3, 2, False),
], ids=lambda v: getattr(v, "name", str(v)))
def test_pools_alone_fully_connected_first_and_no_bias(model, batch, launches, bias):
    _both_ways(model, batch, 100, launches, False, workloads.batch_input(model, batch, 3), bias)


@pytest.mark.parametrize("model,launches", [(_mixed(), 2), (_ends_in_a_map(), 1), (_pools(7, 75), 1), (_only_fc(), 1)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_infinities_and_nan(model, launches):
    # one image each: +inf, -inf, NaN, an image of the lowest finite value, one of zeros, and an ordinary one between
    # the others, which has to stay finite
    x = workloads.batch_input(model, 6, 3)
    C, H, W = model.in_shape
    x[0, 1, 0, 0] = float("inf")
    x[1, C - 1, H - 1, W - 1] = -float("inf")
    x[2, 0, H // 2, W // 2] = float("nan")
    x[3] = -3.3895e38
    x[5] = 0.0
    for t in _both_ways(model, 6, 100, launches, False, x):
        assert t[4].isfinite().all() and t[5].isfinite().all()


def test_an_output_inside_the_input():
    # separate launches: the first layer has read the whole batch before the last one stores
    model, batch = workloads.lenet5(), 40
    dm = lowering.DeviceModel(model, workloads.parameters(model, 4), DEV)
    with gpulet.Partition(0, 100, 0) as p:
        xd = dm.input_to_device(workloads.batch_input(model, batch, 4))
        want, _ = dm.run(p, xd)
        ws, n = dm.workspace(batch)
        over = xd.view(torch.float32).flatten()[:want.numel()]
        before = p.kernel_launches()
        torch.cuda.synchronize()
        gpulet.run_model(dm.desc, batch, p, xd, over, ws, n)
        p.sync()
        assert p.kernel_launches() - before == dm.desc.n_layers
        assert torch.equal(over.view_as(want), want)
