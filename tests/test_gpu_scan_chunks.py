"""Prefix sum across work-groups: chunks of one and of several tiles, partial
last tiles and chunks, rows and arrays that start at 4-byte boundaries only,
in place and not, with exactly the scratch that is asked for.  Values span the
whole 32-bit range, so sums wrap; results are compared bit for bit with
numpy's wrapping cumulative sum.
"""
import numpy as np
import pytest
import torch

from paper_1907_02154_amd import vision

pytestmark = pytest.mark.gpu

TILE = 4096
CASES = [
    # rows, n, offset of x and y in elements
    (1, 5, 1), (3, 1026, 0), (2, TILE + 2, 3),                       # one work-group per row
    (1, 4 * TILE + 1, 0), (1, 4 * TILE + 2, 1), (63, 4 * TILE + 3, 2),   # one tile per chunk
    (1, 1024 * TILE, 0), (1, 1024 * TILE + 1, 1),                    # the most chunks of one tile; two per chunk
    (1, 2048 * TILE + 3 * TILE + 2, 0), (3, 1500 * TILE - 1, 3),     # a last chunk that is not whole; unaligned rows
]


@pytest.mark.parametrize("rows,n,shift", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_scan_chunks(rows, n, shift):
    print("scan", rows, n, shift, flush=True)
    rng = np.random.default_rng(rows + n + shift)
    x = rng.integers(-2**31, 2**31, (rows, n), dtype=np.int64).astype(np.int32)
    incl = np.cumsum(x, axis=1, dtype=np.int32)
    excl = np.concatenate([np.zeros((rows, 1), np.int32), incl[:, :-1]], axis=1)
    guard = 64
    buf = torch.full((rows * n + shift + guard,), 7, dtype=torch.int32, device="cuda")
    out = torch.full_like(buf, 9)
    tx, ty = (t[shift:shift + rows * n].view(rows, n) for t in (buf, out))
    tx.copy_(torch.from_numpy(x))
    need = vision.scan_workspace_bytes(rows, n)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    for exclusive, want in ((False, incl), (True, excl)):
        for rep in range(2):
            vision.scan_i32(tx, ty, exclusive=exclusive, ws=ws)
            np.testing.assert_array_equal(ty.cpu().numpy(), want)
    assert bool((out[:shift] == 9).all()) and bool((out[shift + rows * n:] == 9).all())
    vision.scan_i32(tx, tx, exclusive=False, ws=ws)
    np.testing.assert_array_equal(tx.cpu().numpy(), incl)
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + rows * n:] == 7).all())
