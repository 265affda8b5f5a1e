"""GPU: fp32 convolutions reducing in (c, r, s) order, whose wavefronts decode
their taps 16 blocks at a time into LDS, against the oracle.

On small integers every fp32 sum is exact, so the result must match bit for
bit: partial last blocks, fewer and more than 16 blocks per wavefront, both
pixel widths, padding larger than the image's border, strides, rectangular
filters, split reductions, and filters of more positions than a bit mask
holds (which decode tap by tap).
"""
import numpy as np
import pytest
import torch

from paper_1907_02154_amd import miconv
from paper_1907_02154_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    miconv.lib()


# (N, C, H, W, K, R, S, stride, pad, groups)
CASES = [
    (5, 100, 55, 57, 120, 3, 3, 2, 1, 1),    # 113 blocks, the last one partial
    (1, 9, 8, 9, 33, 3, 3, 1, 1, 1),         # fewer blocks than wavefronts
    (3, 410, 20, 21, 40, 3, 3, 1, 1, 1),     # more than 16 blocks per wavefront, a partial one
    (1, 1032, 9, 9, 32, 3, 3, 1, 1, 1),      # split
    (30, 21, 60, 58, 70, 3, 3, 1, 1, 1),     # two pixel blocks per wavefront
    (2, 20, 17, 19, 36, 5, 5, 1, 4, 2),      # 25 positions, padding past the filter's half, groups
    (2, 11, 15, 16, 34, 1, 7, 1, 0, 1),      # rectangular
    (2, 6, 12, 13, 34, 4, 7, 3, 3, 1),       # 28 positions, stride 3
    (2, 10, 18, 19, 36, 6, 6, 1, 2, 1),      # 36 positions: no mask
]


@pytest.mark.parametrize("mode", ["plain", "ws", "packed"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_wave_taps_small_int_bitwise(oracle_lib, case, mode):
    N, C, H, W, K, R, S, st, pad, g = case
    seed = 5100 + sum(case)
    x = wl.small_ints((N, C, H, W), -4, 4, seed)
    w = wl.small_ints((K, C // g, R, S), -4, 4, seed + 1)
    b = wl.small_ints((K,), -8, 8, seed + 2)
    want = oracle_lib.conv2d(x, w, b, st, pad, g, True)
    tx, tw, tb = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (x, w, b))
    if mode == "packed":
        y = torch.full(want.shape, float("nan"), device="cuda")
        miconv.PackedFilters(tw, (N, C, H, W), st, pad, g).forward(tx, tb, y, relu=True)
    else:
        y = miconv.conv2d(tx, tw, tb, st, pad, g, True, mode=mode)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(y.cpu().numpy(), want)
