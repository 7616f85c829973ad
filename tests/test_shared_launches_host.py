"""When layers that may share a launch do not: input, output and workspace that overlap, a depth split."""

import pytest

from model_launches import INPUT, WORKSPACE, model_launches, straight  # noqa: F401  (fixture)

SMALL = ((8, 28, 28), straight(("conv", 8, 8, 5, 1, 2), ("max", 8, 2, 2, 0), ("fc", 8 * 14 * 14, 16)),
         [("chain", 3)], [("conv", 1), ("pool", 1), ("fc", 1)])
PAIR = ((128, 56, 56), straight(("dw", 128, 1), ("conv", 128, 128, 1, 1, 0)), [("dwpw", 2)], [("dwconv", 1), ("conv", 1)])
POOL = ((256, 28, 28), straight(("conv", 256, 256, 3, 1, 1), ("max", 256, 2, 2, 0)), [("conv+pool", 2)], [("conv", 1), ("pool", 1)])


def _group():
    # a 1x1 layer to a buffer of its own next to one to the output
    a, b = straight(("conv", 64, 64, 1, 1, 0), ("conv", 64, 64, 1, 1, 0))
    a["group_next"] = 1
    b["in_buf"] = 0
    return (64, 40, 40), [a, b], [("group", 2)], [("conv", 1)] * 2


@pytest.mark.parametrize("case", [SMALL, PAIR, POOL, _group()], ids=["chain", "depthwise", "pool", "group"])
def test_overlapping_buffers_keep_layers_apart(model_launches, case):  # noqa: F811
    # One workgroup of a shared launch may store to the output before another has read the input: buffer numbers tell
    # layers apart, addresses need not.
    shape, layers, shared, separate = case
    batch = 32
    size = 2 * batch * shape[0] * shape[1] * shape[2]

    def ask(**kw):
        return model_launches(256, batch, shape, layers, **kw)
    assert ask() == ask(out_at=INPUT + size) == shared
    for out_at in (INPUT, INPUT + 4096, INPUT + size - 256, INPUT - 256):
        assert ask(out_at=out_at) == separate
    assert ask(out_at=WORKSPACE) == ask(in_at=WORKSPACE) == separate


@pytest.mark.parametrize("C,K,H", [(512, 256, 3), (512, 512, 10), (448, 256, 4)])
def test_a_pointwise_layer_that_splits_its_depth_keeps_its_launch(model_launches, C, K, H):  # noqa: F811
    layers = straight(("dw", C, 1), ("conv", C, K, 1, 1, 0))
    assert model_launches(256, 1, (C, H, H), layers) == [("dwpw", 2)]
    assert model_launches(256, 1, (C, H, H), layers, split_k=8) == [("dwconv", 1), ("conv", 1)]


@pytest.mark.parametrize("cu,N,H,W,K,shared", [
    (256, 1, 150, 150, 64, True), (256, 4, 150, 150, 64, True), (256, 32, 150, 150, 64, False),
    (256, 3, 21, 18, 64, False), (256, 1, 38, 38, 64, False), (64, 8, 9, 50, 128, True), (64, 2, 9, 50, 128, False),
    (128, 3, 56, 56, 256, False),
])
def test_depthwise_pairs_of_32_channels(model_launches, cu, N, H, W, K, shared):  # noqa: F811
    layers = straight(("dw", 32, 1), ("conv", 32, K, 1, 1, 0))
    assert model_launches(cu, N, (32, H, W), layers) == ([("dwpw", 2)] if shared else [("dwconv", 1), ("conv", 1)])
