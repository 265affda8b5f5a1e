"""GPU: bf16 filters packed by whole runs of channels, alone
(pack_krsc_run_kernel) and in one launch with the channel-last copy
(pack_nchw_to_nhwc_bf16_kernel), against numpy's transpose and the oracle.

Packing moves values and nothing else, so both must match bit for bit:
partial runs, several per filter, one to 25 taps, and filters at an odd
2-byte address (which the 16-byte loads cannot take).
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


def bf(bits, shift=0):
    """bf16 bits -> a device tensor `shift` values past 16-byte alignment."""
    t = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)
    buf = torch.zeros(t.numel() + 8, device="cuda", dtype=torch.bfloat16)
    out = buf[shift:shift + t.numel()].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("K,C,R,S", [(5, 8, 2, 1), (3, 40, 3, 3), (7, 64, 3, 3), (6, 136, 5, 5), (2, 72, 1, 7)])
@pytest.mark.parametrize("shift", [0, 1])
def test_pack_runs_bitwise(K, C, R, S, shift):
    w = np.random.default_rng(40 + C + R).integers(0, 1 << 16, (K, C, R, S), dtype=np.uint16)
    tw = bf(w, shift)
    shape = (2, C, 16, 16, K, R, S, 1, 0, 1, 1)
    L = miconv.lib()
    n = L.conv2d_packed_weight_bytes(*shape)
    assert n >= w.nbytes
    packed = torch.full((n // 2,), -1, device="cuda", dtype=torch.int16)
    assert L.conv2d_pack_weights(*shape, tw.data_ptr(), packed.data_ptr(), None) == 0
    torch.cuda.synchronize()
    got = packed.cpu().numpy().view(np.uint16)[:w.size]
    np.testing.assert_array_equal(got, np.transpose(w, (0, 2, 3, 1)).ravel())


# (N, C, H, W, K, R, stride, groups, copy): copies of every read width, filters in
# 64-channel blocks (the first) and in plain KRSC order
CASES = [
    (13, 128, 27, 29, 160, 3, 1, 1, 1),
    (3, 64, 40, 46, 72, 3, 1, 1, 8),
    (3, 192, 22, 46, 70, 3, 2, 2, 4),
    (5, 96, 7, 9, 40, 5, 1, 1, 0),
    (2, 64, 33, 35, 24, 2, 1, 1, 1),
]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:8])))
def test_pack_with_copy_small_int_bitwise(oracle_lib, case, shift):
    N, C, H, W, K, R, st, g, copy = case
    pad = R // 2
    name, launches = miconv.conv2d_describe(N, C, H, W, K, R, R, st, pad, g, "bf16")
    assert name.startswith(f"pack_nchw_to_nhwc_bf16_kernel<{copy}> + igemm_bf16"), name
    assert launches == name.count(" + ") + 1
    x = wl.to_bf16_bits(wl.small_ints((N, C, H, W), -4, 4, 71))
    w = wl.to_bf16_bits(wl.small_ints((K, C // g, R, R), -4, 4, 72))
    b = wl.small_ints((K,), -8, 8, 73)
    y = miconv.conv2d(bf(x), bf(w, shift), torch.from_numpy(b).cuda(), st, pad, g, True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(y.cpu().numpy(), oracle_lib.conv2d_bf16(x, w, b, st, pad, g, True))
