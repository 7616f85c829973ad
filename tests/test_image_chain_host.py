"""Which runs of small layers go out as one launch with a workgroup per image."""

from model_launches import model_launches, straight  # noqa: F401  (fixture)


def test_a_run_of_pools_fits_into_lds_as_a_whole(model_launches):  # noqa: F811
    # 2x2 / stride 2 twice: on 47x159 the tensors alone fill the workgroup's 152 KB of LDS
    two = straight(("max", 8, 2, 2, 0), ("max", 8, 2, 2, 0))
    assert model_launches(256, 1, (8, 47, 159), two) == [("pool", 1)] * 2
    assert model_launches(256, 1, (8, 47, 157), two) == [("chain", 2)]
