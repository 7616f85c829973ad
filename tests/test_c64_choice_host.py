"""From how many pixel tiles per workgroup on the 3x3 kernel that keeps 64-channel filters in registers is taken."""

import pytest

from test_conv_choice_host import launches  # noqa: F401  (fixture)


@pytest.mark.parametrize("cu,N,H,K,kernel", [
    (256, 32, 56, 64, "c64"), (128, 16, 56, 64, "c64"),     # three tiles per workgroup, one filter tile
    (256, 30, 56, 64, "gather"), (128, 8, 56, 64, "gather"),
    (128, 8, 56, 192, "c64"), (256, 4, 112, 128, "gather"), (256, 16, 56, 192, "c64"),
])
def test_from_how_many_tiles_on(launches, cu, N, H, K, kernel):  # noqa: F811
    assert launches([(cu, [(N, 64, H, H, K, 3, 3, 1, 1, 64)])])[0][0][0] == kernel


@pytest.mark.parametrize("cu,N,H,K", [
    (128, 32, 20, 256), (64, 32, 20, 128), (64, 24, 30, 96),     # columns of 16 pixels in rows of 20 and 30
    (64, 32, 56, 128), (64, 4, 56, 192),                          # gathered, few and large tiles cover the layer as well
])
def test_not_where_gathering_is_faster(launches, cu, N, H, K):  # noqa: F811
    assert launches([(cu, [(N, 64, H, H, K, 3, 3, 1, 1, 64)])])[0][0][0] == "gather"
