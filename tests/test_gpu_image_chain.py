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
    params = workloads.parameters(model, 3)
    x = workloads.batch_input(model, batch, 3)
    dm = lowering.DeviceModel(model, params, DEV, reuse=reuse)
    with gpulet.Partition(0, pct, 0) as p:
        xd = dm.input_to_device(x)
        tensors = {}
        for fused in (False, True):
            gpulet.set_conv_pool_fusion(fused)
            try:
                before = p.kernel_launches()
                ws, _ = dm.workspace(batch)
                ws.zero_()
                y, _ = dm.run(p, xd)
                assert p.kernel_launches() - before == (launches if fused else dm.desc.n_layers)
            finally:
                gpulet.set_conv_pool_fusion(True)
            named = [] if reuse else [nd.dst for nd in model.nodes if nd.dst != model.out]
            tensors[fused] = [y.clone()] + [dm.read_tensor(t, batch) for t in named]
    for a, b in zip(*tensors.values()):
        assert torch.equal(a, b)


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
