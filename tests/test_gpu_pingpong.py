"""GPU: bf16 3x3 stride-1 layers on the kernel of two alternating wavefront
groups (igemm_bf16_pp_kernel), against the oracle.

On small integers every fp32 sum is exact, whatever its order, so the result
must match bit for bit: an odd number of chunks (the groups' shares differ),
ragged pixel and filter tiles, planes up to the widest patch and down to one
pixel, groups, split reductions with a shorter last part, residuals, and an
fp32 y that 16-byte stores cannot take.
"""
import numpy as np
import pytest
import torch

from paper_1907_02154_amd import miconv
from paper_1907_02154_amd import workloads as wl

pytestmark = pytest.mark.gpu

CL = miconv.LAYOUT_X_NHWC | miconv.LAYOUT_Y_NHWC_BF16


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    miconv.lib()


def bf(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)


def nhwc(a):
    return np.ascontiguousarray(np.transpose(a, (0, 2, 3, 1)))


# (N, C, H, W, K, groups, reduction split)
CASES = [
    (13, 192, 29, 31, 136, 1, False),    # 27 chunks, ragged pixel and filter tiles
    (8, 128, 40, 46, 200, 1, False),     # the widest patch
    (10, 256, 20, 23, 384, 2, False),    # two groups, ragged filter tiles
    (13, 128, 27, 29, 160, 1, False),    # odd plane: scalar stores of an fp32 y
    (12600, 128, 1, 1, 128, 1, False),   # only the middle tap is inside
    (2111, 128, 3, 2, 128, 1, False),
    (47, 512, 7, 7, 512, 1, True),       # parts of three, three and two channel blocks; odd M
    (64, 384, 7, 7, 384, 1, True),       # three parts of two
]


@pytest.mark.parametrize("cl", [True, False], ids=["cl", "nchw"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:6])))
def test_pingpong_small_int_bitwise(oracle_lib, case, cl):
    N, C, H, W, K, g, split = case
    seed = 9300 + sum(case)
    x = wl.to_bf16_bits(wl.small_ints((N, C, H, W), -4, 4, seed))
    w = wl.to_bf16_bits(wl.small_ints((K, C // g, 3, 3), -4, 4, seed + 1))
    b = wl.small_ints((K,), -8, 8, seed + 2)
    res = wl.small_ints((N, K, H, W), -60, 60, seed + 3)
    conv = oracle_lib.conv2d_bf16(x, w, b, 1, 1, g, False)
    tw, tb = bf(w), torch.from_numpy(b).cuda()
    tx = bf(nhwc(x)) if cl else bf(x)
    tres = bf(nhwc(wl.to_bf16_bits(res))) if cl else torch.from_numpy(res).cuda()
    for relu, with_res in ((False, False), (True, True)):
        want = conv + res if with_res else conv
        want = np.maximum(want, 0) if relu else want
        if cl:
            want = nhwc(wl.to_bf16_bits(want))
            y = torch.full((N, H, W, K), float("nan"), device="cuda", dtype=torch.bfloat16)
        else:
            y = torch.full((N, K, H, W), float("nan"), device="cuda")
        s = miconv.Stack([(miconv.OP_CONV_BF16, tx, tw, tb, y, 1, 1, g, relu, tres if with_res else None)
                          + ((CL,) if cl else ())])
        name = s.describe(0)
        assert f"igemm_bf16_pp_kernel<{'true' if cl else 'false'}>" in name, name
        assert ("splitk_reduce" in name) == split, name
        s.launch()
        torch.cuda.synchronize()
        got = y.view(torch.int16).cpu().numpy().view(np.uint16) if cl else y.cpu().numpy()
        np.testing.assert_array_equal(got, want, err_msg=f"relu={relu} res={with_res}")
        s.close()
    if not cl:
        # one float past 16-byte alignment, images further apart than their size
        gap = K * H * W + 3
        buf = torch.full((N * gap + 1,), float("nan"), device="cuda")
        y = buf[1:].as_strided((N, K, H, W), (gap, H * W, W, 1))
        miconv.conv2d_fwd_ws(tx, tw, tb, y, 1, 1, g, False)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(y.cpu().numpy(), conv)
        assert torch.isnan(buf[0]) and torch.isnan(buf[1:].view(N, gap)[:, K * H * W:]).all()
