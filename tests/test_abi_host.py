"""Host-side checks of the C-ABI library (no GPU needed).

The library must load, export every function ``include/miconv.h`` and
``include/mivision.h`` declare,
and reject invalid arguments before any HIP call (so these run on a machine
without a GPU).  The fake pointers below are never dereferenced: every call
here fails validation first.
"""
import ctypes

import pytest

from paper_1907_02154_amd import miconv

FAKE = 4096   # aligned, non-null, never touched


@pytest.fixture(scope="module")
def L():
    return miconv.lib()


def test_exports_every_declared_symbol(L):
    names = miconv.header_functions()
    for expected in ("conv2d_fwd", "conv2d_fwd_bf16", "dwconv2d_fwd", "conv2d_fwd_algo",
                     "conv2d_workspace_bytes", "conv2d_fwd_ws",
                     "miconv_out_dims", "maxpool2d_fwd", "add_act_fwd", "cast_f32_to_bf16",
                     "miconv_strerror", "miconv_last_hip_error", "miconv_version",
                     "vision_scan_i32", "vision_segmented_argsort", "vision_box_nms"):
        assert expected in names
    for n in names:
        assert hasattr(L, n), n


def test_out_dims(L):
    assert miconv.out_dims(224, 224, 7, 7, 2, 3) == (112, 112)
    assert miconv.out_dims(112, 112, 3, 3, 2, 1) == (56, 56)
    assert miconv.out_dims(14, 14, 1, 1, 2, 0) == (7, 7)
    assert miconv.out_dims(5, 6, 3, 2, 2, 0) == (2, 3)
    P, Q = ctypes.c_int(), ctypes.c_int()
    assert L.miconv_out_dims(2, 2, 3, 3, 1, 0, ctypes.byref(P), ctypes.byref(Q)) == miconv.ERR_SHAPE
    assert L.miconv_out_dims(2, 2, 3, 3, 0, 0, ctypes.byref(P), ctypes.byref(Q)) == miconv.ERR_SHAPE
    assert L.miconv_out_dims(2, 2, 3, 3, 1, 0, None, None) == miconv.ERR_NULL


def _call(L, fn, N=1, C=4, H=8, W=8, K=4, R=3, S=3, stride=1, pad=1, groups=1,
          x=FAKE, w=FAKE, b=None, y=FAKE):
    return getattr(L, fn)(N, C, H, W, K, R, S, stride, pad, groups, x, w, b, y, 0, None)


@pytest.mark.parametrize("fn", ["conv2d_fwd", "conv2d_fwd_bf16", "dwconv2d_fwd"])
def test_validation_errors(L, fn):
    assert _call(L, fn, x=None) == miconv.ERR_NULL
    assert _call(L, fn, w=None) == miconv.ERR_NULL
    assert _call(L, fn, y=None) == miconv.ERR_NULL
    for bad in (dict(N=0), dict(C=-1), dict(H=0), dict(W=0), dict(K=0), dict(R=0), dict(S=0),
                dict(stride=0), dict(pad=-1), dict(H=2, W=2, pad=0)):
        assert _call(L, fn, **bad) == miconv.ERR_SHAPE, bad
    assert _call(L, fn, groups=3) == miconv.ERR_GROUPS
    assert _call(L, fn, groups=0) == miconv.ERR_GROUPS
    assert _call(L, fn, N=70000, C=1024, H=64, W=64, K=4, groups=1) == miconv.ERR_TOO_LARGE
    assert _call(L, fn, x=FAKE + 1) == miconv.ERR_ALIGN
    assert _call(L, fn, y=FAKE + 2) == miconv.ERR_ALIGN


def test_depthwise_specific_errors(L):
    assert _call(L, "dwconv2d_fwd", groups=1) == miconv.ERR_GROUPS
    assert _call(L, "dwconv2d_fwd", C=4, K=8, groups=4) == miconv.ERR_GROUPS
    assert _call(L, "dwconv2d_fwd", C=4, K=4, groups=4, R=9, S=9, pad=4) == miconv.ERR_UNSUPPORTED


def test_algo_and_glue_errors(L):
    assert L.conv2d_fwd_algo(1, 4, 8, 8, 4, 3, 3, 1, 1, 1, FAKE, FAKE, None, FAKE, 0, 7, None) == \
        miconv.ERR_UNSUPPORTED
    assert L.maxpool2d_fwd(1, 1, 4, 4, 2, 2, 2, 2, FAKE, FAKE, None) == miconv.ERR_SHAPE   # pad >= R
    assert L.maxpool2d_fwd(1, 1, 4, 4, 2, 2, 2, 0, None, FAKE, None) == miconv.ERR_NULL
    assert L.add_act_fwd(-1, FAKE, FAKE, FAKE, 1, None) == miconv.ERR_SHAPE
    assert L.add_act_fwd(4, None, FAKE, FAKE, 1, None) == miconv.ERR_NULL
    assert L.cast_f32_to_bf16(4, FAKE, FAKE + 1, None) == miconv.ERR_ALIGN


def test_strerror_and_version(L):
    for s in range(0, -9, -1):
        assert miconv.strerror(s) != "unknown status", s
    assert miconv.strerror(-99) == "unknown status"
    assert L.miconv_version() >= 20000
    assert L.miconv_last_hip_error() == 0


def test_packed_weight_sizes(L):
    """Packed filter sizes follow the layout of the kernel each shape takes:
    wave order (fp32: [groups][K/32][Kred/8][64 lanes][4]), KRSC (bf16 3x3),
    tap pairs (bf16 7x7 stem: [K][28][8]); 0 when the kernel reads w as given."""
    f = L.conv2d_packed_weight_bytes
    assert f(1, 64, 56, 56, 64, 3, 3, 1, 1, 1, 0) == 2 * 72 * 256 * 4          # fp32 wave, Kred 576
    assert f(1, 64, 56, 56, 256, 1, 1, 1, 0, 1, 0) == 8 * 8 * 256 * 4          # fp32 wave, Kred 64
    assert f(64, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1) == 64 * 64 * 9 * 2          # bf16 KRSC
    assert f(64, 3, 224, 224, 64, 7, 7, 2, 3, 1, 1) == 64 * 28 * 8 * 2         # bf16 stem
    assert f(64, 256, 56, 56, 64, 1, 1, 1, 0, 1, 1) == 0                       # bf16 1x1: w as given
    assert f(1, 32, 56, 56, 32, 3, 3, 1, 1, 32, 0) == 0                        # depthwise
    assert f(1, 64, 56, 56, 64, 3, 3, 1, 1, 1, 2) == miconv.ERR_UNSUPPORTED    # no such dtype
    assert f(0, 64, 56, 56, 64, 3, 3, 1, 1, 1, 0) == miconv.ERR_SHAPE
    assert f(1, 64, 56, 56, 64, 3, 3, 1, 1, 3, 0) == miconv.ERR_GROUPS


def test_packed_entry_points_validate_first(L):
    shape = (1, 64, 56, 56, 64, 3, 3, 1, 1, 1, 0)
    assert L.conv2d_pack_weights(*shape, None, FAKE, None) == miconv.ERR_NULL
    assert L.conv2d_pack_weights(*shape, FAKE, None, None) == miconv.ERR_NULL
    assert L.conv2d_pack_weights(*shape[:-1], 5, FAKE, FAKE, None) == miconv.ERR_UNSUPPORTED
    assert L.conv2d_fwd_packed(*shape, None, FAKE, None, FAKE, 0, None) == miconv.ERR_NULL
    assert L.conv2d_fwd_packed(*shape, FAKE, None, None, FAKE, 0, None) == miconv.ERR_NULL
    assert L.conv2d_fwd_packed(*shape[:-1], 7, FAKE, FAKE, None, FAKE, 0, None) == miconv.ERR_UNSUPPORTED
    assert L.conv2d_fwd_packed(1, 64, 56, 56, 64, 3, 3, 0, 1, 1, 0, FAKE, FAKE, None, FAKE, 0,
                               None) == miconv.ERR_SHAPE


def test_residual_entry_point_validates_first(L):
    """conv2d_fwd_res checks dtype, pointers, the residual's alignment and the
    operator kind before anything is launched (no GPU needed)."""
    shape = (1, 64, 56, 56, 64, 3, 3, 1, 1, 1)
    A = miconv.ALGO_AUTO
    assert L.conv2d_fwd_res(*shape, 2, A, FAKE, FAKE, None, FAKE, FAKE, 0, None) == miconv.ERR_UNSUPPORTED
    assert L.conv2d_fwd_res(*shape, 0, A, None, FAKE, None, FAKE, FAKE, 0, None) == miconv.ERR_NULL
    assert L.conv2d_fwd_res(*shape, 1, A, FAKE, FAKE, None, FAKE, None, 0, None) == miconv.ERR_NULL
    assert L.conv2d_fwd_res(*shape, 0, 9, FAKE, FAKE, None, FAKE, FAKE, 0, None) == miconv.ERR_UNSUPPORTED
    for off in (2, 4, 8, 12):   # not at y's offset modulo 16 bytes
        assert L.conv2d_fwd_res(*shape, 0, A, FAKE, FAKE, None, FAKE + off, FAKE, 0,
                                None) == miconv.ERR_ALIGN, off
    dw = (1, 32, 28, 28, 32, 3, 3, 1, 1, 32)
    assert L.conv2d_fwd_res(*dw, 0, A, FAKE, FAKE, None, FAKE, FAKE, 0, None) == miconv.ERR_UNSUPPORTED


def test_output_stride_validation(L):
    """conv2d_fwd_ex: the image stride of y must keep images apart, fit 32-bit
    offsets, and is refused for depthwise shapes; checked before any launch."""
    shape = (2, 64, 56, 56, 64, 3, 3, 1, 1, 1)
    A = miconv.ALGO_AUTO
    dense = 64 * 56 * 56
    assert L.conv2d_fwd_ex(*shape, 0, A, FAKE, FAKE, None, None, FAKE, dense - 1, 0, None) == miconv.ERR_SHAPE
    assert L.conv2d_fwd_ex(*shape, 0, A, FAKE, FAKE, None, None, FAKE, 1 << 31, 0, None) == miconv.ERR_TOO_LARGE
    dw = (2, 32, 28, 28, 32, 3, 3, 1, 1, 32)
    assert L.conv2d_fwd_ex(*dw, 0, A, FAKE, FAKE, None, None, FAKE, 64 * 28 * 28, 0, None) == miconv.ERR_UNSUPPORTED
    assert L.conv2d_fwd_ex(*shape, 3, A, FAKE, FAKE, None, None, FAKE, 0, 0, None) == miconv.ERR_UNSUPPORTED


def test_workspace_query(L):
    """conv2d_workspace_bytes: 0 where the fastest plan needs no scratch,
    the split partials / channel-last copy / packed filters otherwise, and
    the validation errors of the conv entry points."""
    f = miconv.conv2d_workspace_bytes
    assert f(1, 1, 1, 1, 1, 1, 1, 1, 0) == 0                                   # one tap
    assert f(1, 512, 7, 7, 512, 3, 3, 1, 1) >= 2 * 512 * 49 * 4               # split partials
    # bf16 3x3 at batch 64: the channel-last copy of x and the KRSC filters
    assert f(64, 128, 28, 28, 128, 3, 3, 1, 1, dtype="bf16") >= 64 * 128 * 28 * 28 * 2 + 128 * 128 * 9 * 2
    with pytest.raises(miconv.MiconvError):
        f(1, 64, 56, 56, 64, 3, 3, 1, 1, groups=3)
    g = L.conv2d_workspace_bytes
    assert g(1, 64, 56, 56, 64, 3, 3, 1, 1, 1, 2, 0) == miconv.ERR_UNSUPPORTED   # dtype
    assert g(1, 64, 56, 56, 64, 3, 3, 1, 1, 1, 0, 9) == miconv.ERR_UNSUPPORTED   # algo
    assert g(0, 64, 56, 56, 64, 3, 3, 1, 1, 1, 0, 0) == miconv.ERR_SHAPE


def test_ws_entry_point_checks_the_workspace_first(L):
    """A plan that needs scratch refuses a missing, short or unaligned
    workspace before anything is enqueued (no GPU needed)."""
    shape = (1, 512, 7, 7, 512, 3, 3, 1, 1, 1)
    need = L.conv2d_workspace_bytes(*shape, 0, 0)
    assert need > 0
    A = miconv.ALGO_AUTO
    call = lambda ws, n: L.conv2d_fwd_ws(*shape, 0, A, FAKE, FAKE, None, None, FAKE, 0, 0, ws, n, None)
    assert call(None, 0) == miconv.ERR_WORKSPACE
    assert call(FAKE, need - 1) == miconv.ERR_WORKSPACE
    assert call(FAKE + 16, need) == miconv.ERR_WORKSPACE      # not 256-byte aligned
    assert L.conv2d_fwd_ws(*shape, 0, A, None, FAKE, None, None, FAKE, 0, 0, FAKE, need, None) == miconv.ERR_NULL
    assert L.conv2d_fwd_ws(*shape, 2, A, FAKE, FAKE, None, None, FAKE, 0, 0, FAKE, need, None) == \
        miconv.ERR_UNSUPPORTED


def test_ws_alignment_is_checked_where_a_slower_plan_needs_no_workspace(L):
    """An fp32 layer whose fastest plan takes scratch and whose next takes
    none: a workspace that is not 256-byte aligned is refused whatever its
    size, not taken for a missing one."""
    shape = (16, 128, 56, 56, 256, 3, 3, 1, 1, 1)
    need = L.conv2d_workspace_bytes(*shape, 0, 0)
    assert need > 0 and L.conv2d_workspace_bytes(*shape, 0, miconv.ALGO_WAVE) == 0
    A = miconv.ALGO_AUTO
    for n in (need, need - 1, 2 * need, 0):
        assert L.conv2d_fwd_ws(*shape, 0, A, FAKE, FAKE, None, None, FAKE, 0, 0, FAKE + 16, n, None) == \
            miconv.ERR_WORKSPACE, n


SCRATCH_KERNELS = ("splitk_reduce", "nchw_to_nhwc", "pack_")


@pytest.mark.parametrize("config", [1, 2, 3, 4, 5, 6])
def test_plain_plans_need_no_scratch(L, config):
    """Every layer of every workload, as the plain entry points plan it, runs
    without split partials, a channel-last copy or a filter-packing launch:
    one kernel, reading only the caller's tensors.  The stack plans of the
    same layers pack nothing per pass either."""
    from paper_1907_02154_amd import workloads as wl
    wk = wl.workload(config)
    dt = "bf16" if wk.dtype == "bf16" else "f32"
    for l in wk.layers:
        if l.kind == "dw":
            continue
        name, n = miconv.conv2d_describe(l.N, l.C, l.H, l.W, l.K, l.R, l.S, l.stride, l.pad, l.groups,
                                         dt, mode="plain")
        assert n == 1 and not any(k in name for k in SCRATCH_KERNELS), (l.name, name)
        name, n = miconv.conv2d_describe(l.N, l.C, l.H, l.W, l.K, l.R, l.S, l.stride, l.pad, l.groups,
                                         dt, mode="packed")
        assert n == 1 and not any(k in name for k in SCRATCH_KERNELS), (l.name, name)
        name, _ = miconv.conv2d_describe(l.N, l.C, l.H, l.W, l.K, l.R, l.S, l.stride, l.pad, l.groups,
                                         dt, mode="stack")
        assert "pack_" not in name, (l.name, name)


def test_no_allocation_or_sync_on_the_call_path():
    """hipMalloc, hipFree and stream/device synchronisation appear only in the
    stack executor's create/destroy, never in the code the conv entry points
    reach."""
    import glob
    import os
    import re
    csrc = os.path.join(os.path.dirname(miconv.__file__), "csrc")
    pat = re.compile(r"\b(hipMalloc\w*|hipFree\w*|hipStreamSynchronize|hipDeviceSynchronize|hipMemset\w*)\s*\(")
    for path in sorted(glob.glob(os.path.join(csrc, "*.hip")) + glob.glob(os.path.join(csrc, "*.h"))):
        with open(path) as f:
            text = f.read()
        hits = pat.findall(text)
        if os.path.basename(path) == "stack.hip":
            body = text[text.index("int miconv_stack_create"):]
            for fn in ("miconv_stack_launch", "miconv_stack_capture", "miconv_stack_replay",
                       "miconv_stack_launch_timed"):
                seg = body[body.index(f"int {fn}("):]
                seg = seg[:seg.index("\n}\n")]
                assert not pat.search(seg), fn
        else:
            assert not hits, (path, hits)


def test_noalloc_rejects_plans_beyond_its_scratch(L):
    """conv2d_fwd_noalloc refuses, before any launch, a plan whose scratch
    exceeds the library's fixed per-GPU array (a bf16 3x3 layer at batch 128
    on 56 x 56 planes stages a 51 MB channel-last copy)."""
    shape = (128, 64, 56, 56, 64, 3, 3, 1, 1, 1)
    assert L.conv2d_workspace_bytes(*shape, 1, 0) > miconv.NOALLOC_SCRATCH_BYTES
    A = miconv.ALGO_AUTO
    assert L.conv2d_fwd_noalloc(*shape, 1, A, FAKE, FAKE, None, None, FAKE, 0, 0, None) == \
        miconv.ERR_WORKSPACE
    assert L.conv2d_fwd_noalloc(*shape, 1, A, None, FAKE, None, None, FAKE, 0, 0, None) == miconv.ERR_NULL


def test_vision_validation(L):
    """The vision entry points reject bad scalars before any HIP call."""
    from paper_1907_02154_amd import vision
    V = vision.lib()
    assert V.vision_scan_workspace_bytes(0, 10) == miconv.ERR_SHAPE
    assert V.vision_scan_workspace_bytes(1, 0) == miconv.ERR_SHAPE
    assert V.vision_scan_workspace_bytes(1 << 16, 1 << 16) == miconv.ERR_TOO_LARGE
    assert V.vision_scan_workspace_bytes(300, 1000) == 0          # one work-group per row: no workspace
    assert V.vision_scan_workspace_bytes(1, 1 << 20) > 0          # across work-groups: tile sums
    assert V.vision_scan_i32(1, 10, None, FAKE, 0, None, 0, None) == miconv.ERR_NULL
    assert V.vision_scan_i32(1, 1 << 20, FAKE, FAKE, 0, None, 0, None) == miconv.ERR_WORKSPACE
    assert V.vision_scan_i32(1, 1 << 20, FAKE, FAKE, 0, FAKE + 16, 1 << 30, None) == miconv.ERR_WORKSPACE
    assert V.vision_argsort_workspace_bytes(0, 1) == miconv.ERR_SHAPE
    assert V.vision_argsort_workspace_bytes(10, 0) == miconv.ERR_SHAPE
    assert V.vision_argsort_workspace_bytes(2048, 1) == 0         # one block: sorted in place in LDS
    assert V.vision_argsort_workspace_bytes(4096, 3) >= 4096 * 24
    assert V.vision_segmented_argsort(100, 1, FAKE, None, 1, FAKE, None, 0, None) == miconv.ERR_NULL
    assert V.vision_segmented_argsort(5000, 1, FAKE, FAKE, 1, FAKE, None, 0, None) == miconv.ERR_WORKSPACE
    assert V.vision_box_nms_workspace_bytes(1, 5000, 6, -1) == miconv.ERR_UNSUPPORTED
    assert V.vision_box_nms_workspace_bytes(1, 5000, 6, 4096) > 0
    assert V.vision_box_nms_workspace_bytes(0, 5000, 6, 400) == miconv.ERR_SHAPE
    nms = lambda **k: V.vision_box_nms(*[k.get(n, d) for n, d in (
        ("B", 1), ("N", 100), ("W", 6), ("data", FAKE), ("out", FAKE), ("ov", 0.5), ("va", 0.0), ("topk", 50),
        ("idx", 0), ("score", 1), ("coord", 2), ("force", 0), ("ws", FAKE), ("wsb", 1 << 30), ("st", None))])
    assert nms(data=None) == miconv.ERR_NULL
    assert nms(coord=3) == miconv.ERR_SHAPE
    assert nms(score=6) == miconv.ERR_SHAPE
    assert nms(idx=6) == miconv.ERR_SHAPE
    assert nms(topk=-1, N=5000) == miconv.ERR_UNSUPPORTED
    assert nms(data=FAKE + 2) == miconv.ERR_ALIGN
    assert nms(ws=None) == miconv.ERR_WORKSPACE
    assert nms(wsb=16) == miconv.ERR_WORKSPACE
