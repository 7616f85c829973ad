"""Which runs of small layers go out as one launch with a workgroup per image."""

from model_launches import model_launches, straight  # noqa: F401  (fixture)


def test_a_run_of_pools_fits_into_lds_as_a_whole(model_launches):  # noqa: F811
    # 2x2 / stride 2 twice: on 47x159 the tensors alone fill the workgroup's 152 KB of LDS
    two = straight(("max", 8, 2, 2, 0), ("max", 8, 2, 2, 0))
    assert model_launches(256, 1, (8, 47, 159), two) == [("pool", 1)] * 2
    assert model_launches(256, 1, (8, 47, 157), two) == [("chain", 2)]


def test_long_rows_keep_a_launch_of_their_own(model_launches):  # noqa: F811
    # from In = 8192 on the fully connected kernel adds in another order than the shared launch's four quarters
    for H, layers in ((64, (("max", 8, 2, 2, 0), ("fc", 8192, 4))), (32, (("conv", 8, 8, 1, 1, 0), ("fc", 8192, 7)))):
        assert ("chain", 2) not in model_launches(256, 1, (8, H, H), straight(*layers))
    assert ("chain", 2) not in model_launches(256, 1, (8192, 1, 1), straight(("fc", 8192, 8), ("fc", 8, 10)))
    assert model_launches(256, 1, (8, 64, 62), straight(("max", 8, 2, 2, 0), ("fc", 8 * 32 * 31, 4))) == [("chain", 2)]
