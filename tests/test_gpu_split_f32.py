"""GPU: fp32 convolutions on the bf16 matrix cores (x and filters split exactly
into three bf16 parts), the path conv2d_fwd_ws and the stack take for fp32
layers bound by the fp32 MFMA rate.

Small integers must match the oracle bit for bit in every tile, with and
without a split reduction; real data must be no further from 64 bits than the
fp32 MFMA kernel; infinities, NaNs and values beyond bf16's largest must come
out as that kernel gives them; a workspace too small for the split copy must
still be served.
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# (N, C, H, W, K, R, stride, pad, groups, kernel, reduction split)
CASES = [
    (5, 75, 58, 46, 288, 3, 1, 1, 3, "igemm_split3_kernel<128, 128, 2, 2, 3>", False),  # half-empty channel blocks
    (4, 100, 36, 49, 67, 5, 1, 2, 1, "igemm_split3_kernel<128, 128, 2, 2, 3>", True),
    (6, 64, 59, 60, 278, 3, 1, 1, 2, "igemm_split3_kernel<256, 64, 4, 1, 2>", False),
    (6, 75, 18, 42, 136, 5, 1, 2, 1, "igemm_split3_kernel<256, 64, 4, 1, 2>", True),
    (4, 74, 59, 40, 282, 3, 1, 0, 2, "igemm_split3_kernel<128, 64, 2, 2, 3>", False),   # no padding
    (4, 64, 54, 50, 276, 5, 2, 0, 1, "igemm_split3_kernel<128, 64, 2, 2, 3>", True),    # 5x5 stride 2
    (5, 75, 55, 42, 273, 3, 1, 0, 3, "igemm_split3_kernel<64, 128, 2, 2, 3>", False),
    (6, 75, 41, 54, 194, 5, 2, 0, 1, "igemm_split3_kernel<64, 128, 2, 2, 3>", True),
    (4, 100, 30, 42, 292, 3, 1, 1, 2, "igemm_split3_kernel<64, 64, 2, 2, 3>", False),
    (1, 75, 58, 39, 188, 5, 1, 0, 1, "igemm_split3_kernel<64, 64, 2, 2, 3>", True),     # one image: 16-byte reduce
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:9])))
@pytest.mark.parametrize("mode", ["ws", "stack"])
def test_split_small_int_bitwise(oracle_lib, case, mode):
    N, C, H, W, K, R, st, pad, g, kernel, split = case
    name = miconv.conv2d_describe(N, C, H, W, K, R, R, st, pad, g, "f32", mode=mode)[0]
    if mode == "ws":
        assert kernel in name and ("splitk_reduce" in name) == split, name
    seed = 7000 + sum(case[:9])
    x = wl.small_ints((N, C, H, W), -3, 3, seed)
    w = wl.small_ints((K, C // g, R, R), -3, 3, seed + 1)
    b = wl.small_ints((K,), -8, 8, seed + 2)
    P, Q = miconv.out_dims(H, W, R, R, st, pad)
    res = wl.small_ints((N, K, P, Q), -50, 50, seed + 3)
    ref = oracle_lib.conv2d(x, w, None, st, pad, g, False)
    join = np.maximum(ref + b[None, :, None, None] + res, 0)   # every sum is exact
    tx, tw, tb = dev(x), dev(w), dev(b)

    def run(xx, y, bias, relu, r):
        if mode == "ws":
            miconv.conv2d_fwd_ws(xx, tw, bias, y, st, pad, g, relu, res=r)
        else:
            s = miconv.Stack([(miconv.OP_CONV_F32, xx, tw, bias, y, st, pad, g, relu, r)])
            s.launch()
            torch.cuda.synchronize()
            s.close()
        torch.cuda.synchronize()
        return y.cpu().numpy()

    y = torch.full((N, K, P, Q), float("nan"), device="cuda")
    np.testing.assert_array_equal(run(tx, y, tb, True, dev(res)), join)
    # x and y at 4-byte offsets, a channel range of a wider tensor, no bias
    xo = torch.empty(tx.numel() + 1, device="cuda")[1:].view(N, C, H, W).copy_(tx)
    wide = torch.full((N, K + 3, P, Q), -7.0, device="cuda")
    np.testing.assert_array_equal(run(xo, wide[:, 1:1 + K], None, False, None), ref)
    assert bool((wide[:, 0] == -7).all()) and bool((wide[:, K + 1:] == -7).all())


def _conv64(x, w, st, pad):
    """One float64 matrix product per tap."""
    N, C, H, W = x.shape
    K, _, R, S = w.shape
    P, Q = miconv.out_dims(H, W, R, S, st, pad)
    xp = torch.nn.functional.pad(x.double(), (pad, pad, pad, pad))
    y = torch.zeros((K, N * P * Q), dtype=torch.float64, device="cuda")
    for r in range(R):
        for s in range(S):
            t = xp[:, :, r:r + (P - 1) * st + 1:st, s:s + (Q - 1) * st + 1:st]
            y += torch.mm(w[:, :, r, s].double(), t.permute(1, 0, 2, 3).reshape(C, -1))
    return y.view(K, N, P, Q).permute(1, 0, 2, 3)


ERR_CASES = [  # (N, C, H, W, K, R, stride): short and long reductions, split and not
    (8, 64, 112, 112, 64, 3, 1), (8, 256, 56, 56, 256, 3, 1), (16, 512, 14, 14, 512, 3, 1), (32, 256, 14, 14, 1024, 1, 1),
    (9, 314, 38, 38, 152, 3, 2), (49, 512, 8, 8, 512, 3, 1),
]


@pytest.mark.parametrize("case", ERR_CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("dist", ["u01", "n01", "tiny"])
def test_split_no_further_from_64_bits(case, dist):
    """The 2-norm error against float64 stays within 1.1 times the fp32 MFMA
    kernel's (both are a few units of fp32 rounding; equal up to noise at
    worst), for non-negative and signed data and for magnitudes whose low
    parts are far down in the exponent range."""
    N, C, H, W, K, R, st = case
    assert "igemm_split3" in miconv.conv2d_describe(N, C, H, W, K, R, R, st, R // 2, 1, "f32")[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(31 + sum(case))
    x = torch.rand((N, C, H, W), generator=g, device="cuda") if dist == "u01" else \
        torch.randn((N, C, H, W), generator=g, device="cuda")
    w = torch.randn((K, C, R, R), generator=g, device="cuda") * (2.0 / (C * R * R)) ** 0.5
    if dist == "tiny":
        x *= 2.0 ** -50
        w *= 2.0 ** -40
    P, Q = miconv.out_dims(H, W, R, R, st, R // 2)
    want = _conv64(x, w, st, R // 2)
    err = {}
    for algo in (miconv.ALGO_AUTO, miconv.ALGO_WAVE):
        y = torch.empty((N, K, P, Q), device="cuda")
        miconv.conv2d_fwd_ws(x, w, None, y, st, R // 2, algo=algo)
        err[algo] = float((y.double() - want).norm() / want.norm())
    assert err[miconv.ALGO_AUTO] <= 1.1 * err[miconv.ALGO_WAVE], err


@pytest.mark.parametrize("case", [CASES[0], CASES[5], CASES[9]], ids=lambda c: "x".join(map(str, c[:9])))
def test_split_non_finite(case):
    """Infinities, NaNs and finite values that round to a bf16 infinity in x
    and w give what the fp32 MFMA kernel gives: the same NaNs and infinities,
    and values equal to fp32 rounding (1e-5 of the sum of magnitudes bounds a
    chain of 2500 sums)."""
    N, C, H, W, K, R, st, pad, g, kernel, _ = case
    rng = np.random.default_rng(5)
    x = rng.uniform(0, 1, (N, C, H, W)).astype(np.float32)
    w = rng.normal(0, 0.05, (K, C // g, R, R)).astype(np.float32)
    for v in (np.inf, -np.inf, np.nan, np.finfo(np.float32).max, -np.finfo(np.float32).max, 1e-42):
        x[rng.integers(N), rng.integers(C), rng.integers(H), rng.integers(W)] = v
    w[3, 0, 0, 0] = np.finfo(np.float32).max      # finite, beyond bf16's largest
    tx, tw = dev(x), dev(w)
    P, Q = miconv.out_dims(H, W, R, R, st, pad)
    got = torch.empty((N, K, P, Q), device="cuda")
    miconv.conv2d_fwd_ws(tx, tw, None, got, st, pad, g)
    want = torch.empty_like(got)
    miconv.conv2d_fwd_ws(tx, tw, None, want, st, pad, g, algo=miconv.ALGO_WAVE)
    mag = torch.empty_like(got)
    miconv.conv2d_fwd_ws(tx.abs(), tw.abs(), None, mag, st, pad, g, algo=miconv.ALGO_WAVE)
    got, want, mag = (t.cpu().numpy() for t in (got, want, mag))
    assert not np.isfinite(want).all()
    fin = np.isfinite(want) & np.isfinite(mag)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.all(np.abs(got[fin] - want[fin]) <= 1e-5 * mag[fin])


def test_split_needs_no_more_scratch_than_given():
    """A workspace that holds the fp32 MFMA kernel's plan but not the split
    copy is served as before, as is the fixed scratch of conv2d_fwd_noalloc,
    bit for bit that kernel's result."""
    N, C, H, W, K = 16, 128, 56, 56, 256
    need = miconv.conv2d_workspace_bytes(N, C, H, W, K, 3, 3, 1, 1)
    small = miconv.conv2d_workspace_bytes(N, C, H, W, K, 3, 3, 1, 1, algo=miconv.ALGO_WAVE)
    assert need > miconv.NOALLOC_SCRATCH_BYTES > small
    x = torch.rand((N, C, H, W), device="cuda")
    w = torch.randn((K, C, 3, 3), device="cuda") * 0.04
    y = [torch.full((N, K, H, W), float("nan"), device="cuda") for _ in range(5)]
    miconv.conv2d_fwd_ws(x, w, None, y[0], 1, 1, algo=miconv.ALGO_WAVE)
    miconv.conv2d_fwd_ws(x, w, None, y[1], 1, 1, ws=miconv.workspace(max(small, 256)))
    miconv.conv2d_fwd_noalloc(x, w, None, y[2], 1, 1)
    miconv.conv2d_fwd_ws(x, w, None, y[3], 1, 1, ws=miconv.workspace(need - 256))
    miconv.conv2d_fwd_ws(x, w, None, y[4], 1, 1, ws=miconv.workspace(need))
    torch.cuda.synchronize()
    for i in (1, 2, 3):
        assert torch.equal(y[i], y[0]), i
    assert not torch.equal(y[4], y[0])
    assert float((y[4] - y[0]).norm() / y[0].norm()) < 2e-6


@pytest.mark.parametrize("case", [CASES[0], CASES[1], CASES[6], CASES[9]], ids=lambda c: "x".join(map(str, c[:9])))
def test_split_non_finite_filters(case):
    """Infinite and NaN filter values give what the fp32 MFMA kernel gives,
    padding included (a tap in the padding is a zero in every kernel, so an
    infinity there is a NaN), and leave every other filter's sums alone (1e-5
    of the sum of magnitudes bounds a chain of 2500 sums)."""
    N, C, H, W, K, R, st, pad, g, kernel, _ = case
    rng = np.random.default_rng(6)
    x = rng.uniform(0.5, 1, (N, C, H, W)).astype(np.float32)
    w = rng.normal(0, 0.05, (K, C // g, R, R)).astype(np.float32)
    # (not among the first taps: the fp32 MFMA kernel may read those past the filter before, times zero)
    w[1, 1, 0, 0], w[2, 3, R // 2, R // 2], w[K // 2, 1, R - 1, 0] = np.inf, -np.inf, np.nan
    w[K - 1, 1, 1, 1], w[K - 1, C // g - 1, 1, 0] = np.inf, -np.inf
    tx, tw = dev(x), dev(w)
    P, Q = miconv.out_dims(H, W, R, R, st, pad)
    got, want, mag = (torch.empty((N, K, P, Q), device="cuda") for _ in range(3))
    assert kernel in miconv.conv2d_describe(N, C, H, W, K, R, R, st, pad, g, "f32")[0]
    miconv.conv2d_fwd_ws(tx, tw, None, got, st, pad, g)
    miconv.conv2d_fwd_ws(tx, tw, None, want, st, pad, g, algo=miconv.ALGO_WAVE)
    miconv.conv2d_fwd_ws(tx, tw.abs(), None, mag, st, pad, g, algo=miconv.ALGO_WAVE)
    got, want, mag = (t.cpu().numpy() for t in (got, want, mag))
    assert np.isinf(want[:, 1]).any() and np.isnan(want[:, K - 1]).all()
    fin = np.isfinite(want)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.all(np.abs(got[fin] - want[fin]) <= 1e-5 * mag[fin])


def test_split_time_does_not_hang_on_the_data():
    """A layer whose input is NaN throughout (a diverged network) is served by
    the fp32 matrix cores after the split products: a few times the usual time
    (the margin of 8 is for a busy machine)."""
    N, C, H, W, K = 8, 256, 56, 56, 256
    w = torch.randn((K, C, 3, 3), device="cuda") * 0.03
    y = torch.empty((N, K, H, W), device="cuda")
    ws = miconv.workspace(miconv.conv2d_workspace_bytes(N, C, H, W, K, 3, 3, 1, 1))
    ms = []
    for x in (torch.rand((N, C, H, W), device="cuda"), torch.full((N, C, H, W), float("nan"), device="cuda")):
        best = 1e9
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            miconv.conv2d_fwd_ws(x, w, None, y, 1, 1, ws=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
    assert bool(torch.isnan(y).all())
    assert ms[1] < 8 * ms[0], ms


@pytest.mark.parametrize("ex,ew", [(-115, 100), (-126, 90), (-138, 95), (100, -118), (90, -140), (-60, -60), (60, 40)],
                         ids=lambda e: "2^%d" % e)
@pytest.mark.parametrize("case", [ERR_CASES[0], ERR_CASES[2], ERR_CASES[4]], ids=lambda c: "x".join(map(str, c)))
def test_split_keeps_every_magnitude(case, ex, ew):
    """x and w far down in fp32's range, subnormal ones included, beside large
    partners: the error against float64 stays within 1.1 times the fp32 MFMA
    kernel's, and is at most the 1e-6 that both show on ordinary data (values
    below 2^-126 are rounded when they are made, which both read alike).
    (-60, -60) has tiny sums, (60, 40) sums beyond 2^80, which are recomputed."""
    N, C, H, W, K, R, st = case
    assert "igemm_split3" in miconv.conv2d_describe(N, C, H, W, K, R, R, st, R // 2, 1, "f32")[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(77 + sum(case))
    x = torch.randn((N, C, H, W), generator=g, device="cuda", dtype=torch.float64).mul_(2.0 ** ex).float()
    w = torch.randn((K, C, R, R), generator=g, device="cuda", dtype=torch.float64).mul_(2.0 ** ew).float()
    P, Q = miconv.out_dims(H, W, R, R, st, R // 2)
    want = _conv64(x, w, st, R // 2)
    err = {}
    for algo in (miconv.ALGO_AUTO, miconv.ALGO_WAVE):
        y = torch.empty((N, K, P, Q), device="cuda")
        miconv.conv2d_fwd_ws(x, w, None, y, st, R // 2, algo=algo)
        err[algo] = float((y.double() - want).norm() / want.norm())
    assert err[miconv.ALGO_AUTO] <= min(1.1 * err[miconv.ALGO_WAVE], 1e-6), err


# kind -> (bits of x, share of x that is not zero, bits of w, share of w): which of the six
# products carry the result besides hi * hi
PART_KINDS = {
    "x_mid": (11, 1.0, 1, 1.0),       # mid * hi
    "w_mid": (1, 1.0, 11, 1.0),       # hi * mid
    "mid_mid": (10, 0.05, 10, 0.05),  # and mid * mid
    "x_lo": (18, 1.0, 1, 0.006),      # lo * hi
    "w_lo": (1, 0.006, 18, 1.0),      # hi * lo
}


def _part_ints(shape, bits, share, rng):
    """Odd integers of up to `bits` bits, a share of them kept: the lowest bit
    is in the lowest part that the size needs (bf16 holds 8 bits, two parts 16)."""
    v = rng.integers(0, 1 << (bits - 1), shape, dtype=np.int64) * 2 + 1
    v *= rng.choice((-1, 1), shape)
    return np.where(rng.random(shape) < share, v, 0).astype(np.float32)


@pytest.mark.parametrize("kind", PART_KINDS)
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:9])))
def test_split_parts_bitwise(oracle_lib, case, kind):
    """Integers that one bf16 cannot hold, with sums of magnitudes below 2^23
    (every order of summation is exact): a part that is swapped, misplaced or
    stale shows in every tile, tail, group, copy and split reduction."""
    N, C, H, W, K, R, st, pad, g, kernel, _ = case
    assert kernel in miconv.conv2d_describe(N, C, H, W, K, R, R, st, pad, g, "f32")[0]
    xb, xs, wb, ws = PART_KINDS[kind]
    rng = np.random.default_rng(1000 + sum(case[:9]))
    x = _part_ints((N, C, H, W), xb, xs, rng)
    w = _part_ints((K, C // g, R, R), wb, ws, rng)
    ref = oracle_lib.conv2d(x, w, None, st, pad, g, False)
    assert oracle_lib.conv2d(np.abs(x), np.abs(w), None, st, pad, g, False).max() < 2 ** 23
    tx, tw = dev(x), dev(w)
    xo = torch.empty(tx.numel() + 1, device="cuda")[1:].view(N, C, H, W).copy_(tx)   # 4-byte reads in the copy
    for xx in (tx, xo):
        y = torch.full(ref.shape, float("nan"), device="cuda")
        miconv.conv2d_fwd_ws(xx, tw, None, y, st, pad, g)
        np.testing.assert_array_equal(y.cpu().numpy(), ref)


@pytest.mark.parametrize("case", ERR_CASES, ids=lambda c: "x".join(map(str, c)))
def test_split_dropped_products_at_their_largest(case):
    """x = w = 0x1.00ff8p0 throughout: the three products that are left out are
    at their largest, 2^-24 of the whole, and all of one sign.  The error
    against float64 is at most that above the fp32 MFMA kernel's."""
    N, C, H, W, K, R, st = case
    v = float.fromhex("0x1.00ff8p0")
    x, w = torch.full((N, C, H, W), v, device="cuda"), torch.full((K, C, R, R), v, device="cuda")
    P, Q = miconv.out_dims(H, W, R, R, st, R // 2)
    want = _conv64(x, w, st, R // 2)
    err = {}
    for algo in (miconv.ALGO_AUTO, miconv.ALGO_WAVE):
        y = torch.empty((N, K, P, Q), device="cuda")
        miconv.conv2d_fwd_ws(x, w, None, y, st, R // 2, algo=algo)
        err[algo] = float((y.double() - want).norm() / want.norm())
    assert err[miconv.ALGO_AUTO] <= 1.1 * err[miconv.ALGO_WAVE] + 2.0 ** -24, err
