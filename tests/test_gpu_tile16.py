"""The 16x16 gathering tile, which takes the place of 32x32 where its workgroups all start at once: against the oracle
and bit for bit against the tiles that can be forced."""

import pytest
import torch

from paper_2109_01611_amd import inputs

from gpu_util import assert_conv_close, conv_tensors, gpu_conv
from test_conv_choice_host import launches  # noqa: F401  (fixture)
from test_gpu_layers import part  # noqa: F401  (fixture)

# N, C, H, W, K, k, stride, pad, channels of the destination (0: K), residual
CASES = [
    (1, 512, 7, 7, 96, 1, 1, 0, 0, True),       # 49 rows: a ragged fourth tile; a stage of four slices twice
    (1, 2048, 7, 7, 512, 1, 1, 0, 0, False),    # deep 1x1
    (1, 64, 5, 3, 24, 1, 1, 0, 0, True),        # one slice, ragged filter tile, 15 rows
    (1, 72, 6, 5, 40, 1, 1, 0, 64, False),      # a slice with eight channels only, a slice of a wider tensor
    (1, 40, 9, 7, 21, 3, 2, 1, 0, False),       # stored depth order, filters no multiple of 8 (element-wise stores): 32x32
    (1, 40, 9, 7, 21, 7, 2, 3, 0, False),       # the same with a long depth
    (2, 72, 6, 5, 40, 5, 1, 2, 64, False),      # ... a partial last slice, a slice of a wider tensor
    (2, 128, 9, 9, 40, 3, 2, 1, 0, True),       # taps inside 64-channel blocks, rows that span images
    (1, 64, 12, 12, 24, 7, 2, 3, 0, False),     # more taps than the mask of a pixel row holds
    (1, 320, 4, 4, 16, 1, 2, 0, 0, True),       # strided 1x1, a single tile of 4 rows
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_tile16_parity(part, case):  # noqa: F811
    N, C, H, W, K, k, stride, pad, ct, with_res = case
    x, w, b = conv_tensors(23, N, C, H, W, K, k)
    P, Q = ((e + 2 * pad - k) // stride + 1 for e in (H, W))
    res = inputs.tensor(23, "res_tile16", (N, K, P, Q), "normal") if with_res else None
    off = 8 if ct else 0
    got, raw = gpu_conv(part, x, w, b, stride, pad, True, residual=res, ch_total=ct, ch_offset=off)
    assert_conv_close(got[:, off:off + K], x, w, b, stride, pad, True, residual=res)
    for tile in (14, 3):
        assert torch.equal(raw, gpu_conv(part, x, w, b, stride, pad, True, residual=res, ch_total=ct, ch_offset=off, tile=tile)[1])


def test_tile16_is_what_the_cases_get(launches):  # noqa: F811
    got = launches([(256, [(N, C, H, W, K, k, k, s, p, C)]) for N, C, H, W, K, k, s, p, _, _ in CASES])
    assert [g[0][:2] for g in got] == [("gather", 14 if c[1] % 64 and 1 < c[5] ** 2 < 1792 / c[1] else 15) for c in CASES]
    assert ("gather", 15) in [g[0][:2] for g, c in zip(got, CASES) if c[1] % 64 and c[5] > 1]
    # filters larger than 1x1, channels no multiple of 64, a short depth
    for N, C, H, K, k, s in ((1, 8, 14, 24, 3, 2), (1, 16, 1, 96, 5, 1), (1, 96, 7, 64, 3, 1)):
        assert launches([(160, [(N, C, H, H, K, k, k, s, k // 2, C)])])[0][0][:2] == ("gather", 14)
    # not with more 16x16 tiles than CUs
    assert launches([(64, [(1, 2048, 7, 7, 512, 1, 1, 1, 0, 2048)])])[0][0][:2] == ("gather", 14)
