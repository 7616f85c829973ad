"""Which fully connected layers run in the kernel instance that holds 16 depth steps in flight."""

import pytest

from model_launches import model_launches, straight  # noqa: F401  (fixture)


@pytest.mark.parametrize("cu,N,In,Out,kernel", [
    (256, 1, 2048, 1000, "fc-deep"), (256, 32, 4096, 4096, "fc-deep"), (256, 256, 2048, 1000, "fc-deep"), (64, 1, 2048, 1000, "fc-deep"),
    (256, 1, 2040, 1000, "fc"), (256, 1, 64, 4096, "fc"), (256, 1024, 256, 1000, "fc"),     # no 16 steps per wavefront
    (256, 1024, 2048, 1000, "fc"), (256, 512, 2048, 1000, "fc"), (64, 32, 2048, 4096, "fc"),      # more than two workgroups per CU
    (256, 1, 8192, 1000, "fc"),                                                                  # another kernel
])
def test_deep_instance(model_launches, cu, N, In, Out, kernel):  # noqa: F811
    assert model_launches(cu, N, (In, 1, 1), straight(("fc", In, Out))) == [(kernel, 1)]
