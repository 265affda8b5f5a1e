"""GPU: the vision operators (include/mivision.h) against the oracle
(oracle/vision.py), through the C ABI.

Integer and index results must match bit for bit: the prefix sums, the
argsort's local indices (ties are broken by position on both sides, so the
answer is unique), and box_nms's output, whose kept rows are copies of input
rows and whose every other value is -1.  IoU is evaluated in fp32 with the
same operations in the same order on both sides, so the threshold decisions
agree.  Cases span single and several tiles, ragged tails, the one-row and
across-work-group scan paths, empty and long segments, ties, signed zeros,
NaN and infinite keys, topk limits, classes, force_suppress, no class field,
several images, the largest candidate count, and the SSD-like detection
workload at full size.
"""
import json
import os

import numpy as np
import pytest
import torch

from paper_1907_02154_amd import detections as det
from paper_1907_02154_amd import miconv
from paper_1907_02154_amd import vision

pytestmark = pytest.mark.gpu

GOLD = os.path.join(os.path.dirname(__file__), "golden", "vision_examples.json")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vision.lib()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# ---------------------------------------------------------------- scan

SCAN_CASES = [
    (1, 1), (1, 4095), (1, 4096), (1, 4097), (3, 10000), (1, 16384), (1, 16385),   # one work-group per row
    (2, 100000), (1, 1 << 20), (5, 70001),                                            # across work-groups
    (300, 1000), (64, 20000), (70, 30000),                                             # many rows
]


@pytest.mark.parametrize("rows,n", SCAN_CASES, ids=[f"{r}x{n}" for r, n in SCAN_CASES])
def test_scan_bitwise(oracle_lib, rows, n):
    x = det.scan_values((rows, n), seed=rows * 7 + n)
    assert vision.scan_workspace_bytes(rows, n) >= 0
    tx = dev(x)
    for exclusive in (False, True):
        y = vision.scan_i32(tx, exclusive=exclusive)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        f = oracle_lib.scan_exclusive_i32 if exclusive else oracle_lib.scan_inclusive_i32
        for r in range(rows):
            np.testing.assert_array_equal(got[r], f(x[r]), err_msg=f"row {r} exclusive={exclusive}")


def test_scan_in_place_and_hand_example(oracle_lib):
    with open(GOLD) as f:
        g = json.load(f)["scan"]
    t = dev(np.int32(g["x"]))
    vision.scan_i32(t, t)
    torch.cuda.synchronize()
    assert t.cpu().tolist() == g["inclusive"]
    x = det.scan_values((2, 50000), seed=5)
    t = dev(x)
    vision.scan_i32(t, t, exclusive=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(t.cpu().numpy()[1], oracle_lib.scan_exclusive_i32(x[1]))


# ---------------------------------------------------------------- argsort

def _check_argsort(oracle_lib, keys, off, descending):
    out = vision.segmented_argsort(dev(keys), dev(off), descending)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), oracle_lib.segmented_argsort(keys, off, descending))


ARGSORT_CASES = [   # (n, segments, ties)
    (7, 2, False), (2048, 1, False), (2049, 3, True), (5000, 40, True), (30000, 1, False),
    (100000, 700, False), (100000, 13, True), (262144, 2000, False), (1000, 1000, True),
]


@pytest.mark.parametrize("n,segments,ties", ARGSORT_CASES, ids=[f"{a}-{b}-{c}" for a, b, c in ARGSORT_CASES])
def test_segmented_argsort_bitwise(oracle_lib, n, segments, ties):
    keys = det.keys(n, seed=n + segments, ties=ties)
    off = det.segment_offsets(segments, n, seed=segments)
    for descending in (True, False):
        _check_argsort(oracle_lib, keys, off, descending)


def test_argsort_hand_examples_and_special_keys(oracle_lib):
    with open(GOLD) as f:
        for c in json.load(f)["argsort"]:
            out = vision.segmented_argsort(dev(np.float32(c["keys"])), dev(np.int32(c["offsets"])), c["descending"])
            torch.cuda.synchronize()
            assert out.cpu().tolist() == c["expect"], c
    keys = np.float32([0.0, -0.0, np.inf, -np.inf, np.nan, 1.0, -1.0, np.nan, 0.0, -0.0] * 500)
    off = det.segment_offsets(17, keys.size, seed=3)
    for descending in (True, False):
        _check_argsort(oracle_lib, keys, off, descending)


def test_argsort_positions_past_the_segments():
    """Positions at or past offsets[segments] belong to no segment: -1."""
    keys = det.keys(5000, seed=1)
    off = np.int32([0, 1000, 3000])
    out = vision.segmented_argsort(dev(keys), dev(off)).cpu().numpy()
    assert np.all(out[3000:] == -1)
    assert sorted(out[:1000].tolist()) == list(range(1000))


# Edges of the blocks (2048, 4096 or 8192 elements by size and segments) and of
# the merge passes over them, more segments than a block has positions (most
# of them empty), and the radix passes over few long segments (n >= 500000 for
# one, 1.5 million for more).
ARGSORT_BLOCK_CASES = [   # (n, segments, ties)
    (2047, 1, False), (2048, 5, True), (4096, 1, False), (4097, 2, True), (8192, 8, True), (8193, 1, False),
    (16384, 2, True), (16385, 16385, False), (24577, 3, False), (70000, 1, True), (12000, 40000, False),
    (499999, 1, False), (500000, 1, True), (507904, 1, False), (1500000, 15, True), (1500001, 3, False),
    (1500001, 20, True), (1600000, 900, False),
]


@pytest.mark.parametrize("n,segments,ties", ARGSORT_BLOCK_CASES, ids=[f"{a}-{b}-{c}" for a, b, c in ARGSORT_BLOCK_CASES])
def test_argsort_blocks_and_radix_bitwise(oracle_lib, n, segments, ties):
    keys = det.keys(n, seed=n + segments, ties=ties)
    keys[::97], keys[5::101], keys[7::103] = np.nan, -0.0, np.inf
    off = det.segment_offsets(segments, n, seed=segments)
    for descending in (True, False):
        _check_argsort(oracle_lib, keys, off, descending)
    # the last 300 positions belong to no segment
    cut = np.minimum(off, n - 300).astype(np.int32)
    out = vision.segmented_argsort(dev(keys), dev(cut)).cpu().numpy()
    np.testing.assert_array_equal(out[:n - 300], oracle_lib.segmented_argsort(keys[:n - 300], cut, True))
    assert np.all(out[n - 300:] == -1)


# ---------------------------------------------------------------- box_nms

def _check_nms(oracle_lib, data, **kw):
    got = vision.box_nms(dev(data), **kw)
    torch.cuda.synchronize()
    ref = oracle_lib.box_nms(data, **kw)
    np.testing.assert_array_equal(got.cpu().numpy(), ref)
    return ref


def test_nms_hand_examples(oracle_lib):
    with open(GOLD) as f:
        for c in json.load(f)["nms"]:
            d = np.float32(c["data"])[None]
            _check_nms(oracle_lib, d, overlap_thresh=c["overlap_thresh"], valid_thresh=c["valid_thresh"],
                       topk=c["topk"], force_suppress=c["force_suppress"])


NMS_CASES = [   # (batch, num, topk, force, id_index, thresh)
    (1, 50, -1, False, 0, 0.5),
    (2, 1000, 64, False, 0, 0.45),
    (3, 2000, 65, True, 0, 0.3),
    (1, 4096, -1, False, 0, 0.5),       # the largest candidate count
    (4, 5000, 400, False, -1, 0.45),    # no class field
    (2, 3000, 129, False, 0, 0.0),      # any overlap suppresses
    (1, 700, 0, False, 0, 0.5),         # topk 0: everything invalid
    (2, 30000, 200, False, 0, 0.45),    # candidate flags of a row over two scan tiles
]


@pytest.mark.parametrize("case", NMS_CASES, ids=["-".join(map(str, c)) for c in NMS_CASES])
def test_box_nms_bitwise(oracle_lib, case):
    B, N, topk, force, id_index, thr = case
    data = det.detection_rows(B, N, classes=5, objects=8, seed=N + B, object_frac=0.3)
    if id_index < 0:
        data = np.ascontiguousarray(data[..., 1:])   # [score, x1, y1, x2, y2]
        ref = _check_nms(oracle_lib, data, overlap_thresh=thr, valid_thresh=0.01, topk=topk, id_index=-1,
                         score_index=0, coord_start=1, force_suppress=force)
    else:
        ref = _check_nms(oracle_lib, data, overlap_thresh=thr, valid_thresh=0.01, topk=topk,
                         force_suppress=force)
    kept = np.all(ref != -1, axis=2).sum(axis=1)
    assert kept.min() > 0 if topk != 0 else kept.max() == 0


PICK_CASES = [   # (batch, num, topk, scores): chunks of 1024 rows, ranking by comparing up to 512, else by radix passes
    (3, 1023, 512, "ties"), (2, 1025, 513, "ties"), (1, 1, 5, "plain"), (4, 3000, 64, "ties"), (2, 9000, 4096, "plain"),
    (2, 5000, 400, "inf"), (3, 2500, 100, "nan"), (1, 4096, 4096, "ties"), (2, 700, 1000, "nan"),
]


@pytest.mark.parametrize("case", PICK_CASES, ids=["-".join(map(str, c)) for c in PICK_CASES])
def test_box_nms_pick_bitwise(oracle_lib, case):
    """The best topk of more candidates than that: equal scores at the cut
    (taken in row order), infinite scores, NaN scores (never candidates)."""
    B, N, topk, scores = case
    data = det.detection_rows(B, N, classes=5, objects=8, seed=N + topk, object_frac=0.3)
    u = np.random.default_rng(N).uniform(size=(B, N))
    if scores == "ties":
        data[..., 1] = np.round(data[..., 1] * 8) / 8 + 0.02
    elif scores == "inf":
        data[..., 1] = np.where(u < 0.5, np.inf, data[..., 1])
    elif scores == "nan":
        data[..., 1] = np.where(u < 0.1, np.nan, data[..., 1] - 0.2)
    for valid in (0.01, -1.0):
        _check_nms(oracle_lib, data, overlap_thresh=0.45, valid_thresh=valid, topk=topk)


# B, rows, share of valid rows, distinct scores (0: all differ), topk: images picked through slices
SLICE_CASES = [
    (1, 65536, 1.0, 0, 400),          # the most rows picked at once
    (1, 65537, 1.0, 0, 400),          # one row past it, in a chunk and a slice of its own
    (1, 65537, 1.0, 3, 4096),         # the largest topk; the cut falls among equal scores
    (2, 80000, 1.0, 4, 700),
    (1, 150001, 1.0, 2, 1),
    (1, 200000, 1.0, 5, 1000),        # ties across slices
    (3, 100000, 0.001, 0, 400),       # fewer candidates than topk
    (1, 300000, 0.02, 0, 100),
]


@pytest.mark.parametrize("case", SLICE_CASES)
def test_box_nms_slices_bitwise(oracle_lib, case):
    B, N, share, distinct, topk = case
    rng = np.random.default_rng(N + topk)
    s = rng.random((B, N), dtype=np.float32) * 0.9 + 0.05
    if distinct:
        s = (rng.integers(1, distinct + 1, (B, N)) / np.float32(8)).astype(np.float32)
    s[rng.random((B, N)) >= share] = 0
    if B > 1:
        s[1, : N // 2] = 0            # whole slices without a candidate
    xy = rng.random((B, N, 2), dtype=np.float32)
    wh = rng.random((B, N, 2), dtype=np.float32) * np.float32(0.3)
    data = np.concatenate([rng.integers(0, 2, (B, N, 1)).astype(np.float32), s[..., None], xy, xy + wh], axis=2)
    ref = oracle_lib.vision.box_nms(data, 0.3, 0.01, topk=topk)
    got = vision.box_nms(dev(data), 0.3, 0.01, topk)
    np.testing.assert_array_equal(got.cpu().numpy(), ref)


def test_box_nms_iou_rounding_at_threshold(oracle_lib):
    """4096 images of two same-class boxes whose IoU lies within a few ulps
    of the 0.5 threshold (B is A shifted right by about a third of its
    width): the keep / suppress decision follows the fp32 rounding of every
    product and sum, so a kernel that fused a product into the union's sums
    (one rounding fewer) disagrees with the oracle on some of them."""
    rng = np.random.default_rng(44)
    f = np.float32
    B = 4096
    d = np.zeros((B, 2, 6), np.float32)
    x0, y0 = rng.uniform(0, 1, B).astype(f), rng.uniform(0, 1, B).astype(f)
    w, h = rng.uniform(0.05, 0.5, B).astype(f), rng.uniform(0.05, 0.5, B).astype(f)
    dx = (w / f(3)).astype(f)
    dx = (dx + rng.integers(-3, 4, B).astype(f) * np.spacing(dx)).astype(f)
    d[:, :, 0] = 1
    d[:, 0, 1], d[:, 1, 1] = 0.9, 0.8
    d[:, 0, 2:6] = np.stack([x0, y0, x0 + w, y0 + h], 1)
    d[:, 1, 2:6] = np.stack([x0 + dx, y0, x0 + dx + w, y0 + h], 1)
    ref = _check_nms(oracle_lib, d, overlap_thresh=0.5, valid_thresh=0.0, topk=-1)
    kept2 = np.all(ref[:, 1] != -1, axis=1)
    assert 0 < kept2.sum() < B   # both decisions occur


def test_box_nms_detection_workload(oracle_lib):
    """The SSD-like workload at full size: 24564 rows per image, 20 classes,
    scores above 0.01, the best 400 compared, IoU threshold 0.45; one image
    and a batch of 4."""
    for B in (1, 4):
        data = det.detection_rows(B, seed=B)
        ref = _check_nms(oracle_lib, data, overlap_thresh=0.45, valid_thresh=0.01, topk=400)
        kept = np.all(ref != -1, axis=2).sum(axis=1)
        assert kept.min() >= 5 and kept.max() < 400


def test_box_nms_repeated_calls_share_workspace(oracle_lib):
    """A second call on the same workspace (left holding the first call's
    state) with a smaller input gives the second input's answer."""
    ws = miconv.workspace(vision.box_nms_workspace_bytes(2, 3000, 6, 300))
    d1 = det.detection_rows(2, 3000, seed=21, object_frac=0.3)
    d2 = det.detection_rows(1, 1000, seed=22, object_frac=0.3)
    for d in (d1, d2):
        got = vision.box_nms(dev(d), 0.45, 0.01, 300, ws=ws)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), oracle_lib.box_nms(d, 0.45, 0.01, 300))


def test_box_nms_graph_capture_replays(oracle_lib):
    """The whole pipeline captured into a HIP graph on its first call and
    replayed: every replay equals the oracle."""
    d = dev(det.detection_rows(2, 6000, seed=9, object_frac=0.2))
    ref = oracle_lib.box_nms(d.cpu().numpy(), 0.45, 0.01, 256)
    out = torch.empty_like(d)
    ws = miconv.workspace(vision.box_nms_workspace_bytes(2, 6000, 6, 256))
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            vision.box_nms(d, 0.45, 0.01, 256, out=out, ws=ws)
    for rep in range(3):
        out.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), ref, err_msg=f"replay {rep}")


def test_vision_rejections():
    d = torch.zeros((1, 10, 6), device="cuda")
    with pytest.raises(miconv.MiconvError) as e:
        vision.box_nms(d, coord_start=3)
    assert e.value.status == miconv.ERR_SHAPE
    with pytest.raises(miconv.MiconvError) as e:
        vision.box_nms(torch.zeros((1, 5000, 6), device="cuda"), topk=-1)
    assert e.value.status == miconv.ERR_UNSUPPORTED
