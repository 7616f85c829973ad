"""Which runs of small layers go out as one launch with a workgroup per image."""

import pytest

from model_launches import model_launches, straight  # noqa: F401  (fixture)


def test_a_run_of_pools_fits_into_lds_as_a_whole(model_launches):  # noqa: F811
    # seven 3x3 / stride 1 pools on 16x76: the eight tensors alone fill the workgroup's 152 KB of LDS
    seven = straight(*[("max", 8, 3, 1, 1)] * 7)
    assert model_launches(256, 1, (8, 16, 76), seven) == [("chain", 6), ("pool", 1)]
    assert model_launches(256, 1, (8, 16, 75), seven) == [("chain", 7)]


def test_long_rows_keep_a_launch_of_their_own(model_launches):  # noqa: F811
    # from In = 8192 on the fully connected kernel adds in another order than the shared launch's four quarters
    for H, W, layers in ((64, 64, (("max", 8, 2, 2, 0), ("fc", 8192, 4), ("fc", 4, 2))),
                         (32, 32, (("conv", 8, 8, 1, 1, 0), ("fc", 8192, 7), ("fc", 7, 8)))):
        assert len(model_launches(256, 1, (8, H, W), straight(*layers))) == 3
    assert ("chain", 2) not in model_launches(256, 1, (8192, 1, 1), straight(("fc", 8192, 8), ("fc", 8, 10)))
    assert model_launches(256, 1, (8, 64, 62), straight(("max", 8, 2, 2, 0), ("fc", 8 * 32 * 31, 4), ("fc", 4, 2))) == [("chain", 3)]


LENET = straight(("conv", 8, 8, 5, 1, 2), ("max", 8, 2, 2, 0), ("conv", 8, 16, 5, 1, 0), ("max", 16, 2, 2, 0), ("fc", 400, 120),
                 ("fc", 120, 84), ("fc", 84, 10))


@pytest.mark.parametrize("cu", [64, 128, 256])
def test_lenet_is_one_launch_at_every_batch(model_launches, cu):  # noqa: F811
    for batch in (1, 32, 300, 2048):
        assert model_launches(cu, batch, (8, 28, 28), LENET) == [("chain", 7)]


# where one CU per image is the slower way (us, separate launches and one)
@pytest.mark.parametrize("cu,batch,shape,layers", [
    (256, 1, (256, 7, 7), (("conv", 256, 64, 1, 1, 0), ("conv", 64, 256, 1, 1, 0))),        # 7.3 and 13.7
    (256, 2048, (256, 7, 7), (("conv", 256, 64, 1, 1, 0), ("conv", 64, 256, 1, 1, 0))),     # 30 and 102
    (256, 4, (24, 28, 28), (("conv", 24, 24, 3, 1, 1), ("conv", 24, 24, 3, 1, 1))),         # 8.5 and 15.1
    (256, 2048, (256, 1, 1), (("fc", 256, 256), ("fc", 256, 32))),                          # 10.6 and 60
    (256, 512, (8, 48, 48), (("max", 8, 2, 2, 0), ("max", 8, 2, 2, 0))),                    # 7.7 and 10.4
    (64, 256, (16, 7, 7), (("conv", 16, 48, 1, 1, 0), ("conv", 48, 48, 1, 1, 0), ("conv", 48, 96, 1, 1, 0))),
])
def test_wide_layers_and_short_runs_of_many_images_are_not(model_launches, cu, batch, shape, layers):  # noqa: F811
    assert len(model_launches(cu, batch, shape, straight(*layers))) == len(layers)
