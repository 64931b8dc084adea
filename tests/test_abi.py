"""Host-side checks of the C ABI: symbols, argument validation, behaviour with no GPU (CPU only)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
from paper_2407_02327_amd import qsync          # fails loudly when the library is missing or does not load
lib = qsync.lib
P = ctypes.c_void_p
A = P(4096)            # a non-NULL, 16-byte aligned fake device address: validation never dereferences
U = P(4100)            # misaligned


def _gpu_visible() -> bool:
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


# Several tests end with a well-formed call on the fake addresses above, expecting "OK or launch failed": with a GPU
# present such a launch would dereference them, so the whole module runs only where there is none.
pytestmark = pytest.mark.skipif(_gpu_visible(), reason="argument validation on fake device addresses: CPU-only boxes")


def test_every_declared_symbol_is_exported():
    inc = os.path.join(ROOT, "include")
    headers = sorted(f for f in os.listdir(inc) if f.endswith(".h"))
    assert "qsync.h" in headers
    header = "\n".join(open(os.path.join(inc, f)).read() for f in headers)
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = set(re.findall(r"\b(qsync_[a-z0-9_]+)\s*\(", header))
    assert {"qsync_absmax_scale", "qsync_quantize", "qsync_qlinear_fwd", "qsync_qlinear_bwd",
            "qsync_dequantize"} <= names
    for n in names:
        assert hasattr(lib, n), n
        assert n in qsync.SIGNATURES, f"binding lacks {n}"


def test_strerror_and_version():
    assert lib.qsync_version() >= 100
    for s in range(0, -8, -1):
        assert lib.qsync_strerror(s)
    assert b"unknown" in lib.qsync_strerror(-99)


def test_absmax_validation():
    g = lib.qsync_absmax_scale
    f = lambda *a: g(*a[:10], None, None, *a[10:])        # colsum_opt and sumsq_opt absent
    assert f(None, 0, 4, 4, 4, 0, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_NULL
    assert f(A, 0, 4, 4, 4, 0, 8, None, A, None, A, 1 << 20, None) == qsync.ERR_NULL
    assert f(A, 7, 4, 4, 4, 0, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_BAD_ENUM
    assert f(A, qsync.I8, 4, 4, 4, 0, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 4, 4, 4, 3, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, -1, 4, 4, 0, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 4, 4, 3, 0, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 1 << 40, 1 << 40, 1 << 40, 0, 8, A, A, None, A, 1 << 20, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 4, 4, 4, 0, 9, A, A, None, A, 1 << 20, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 4, 4, 4, 0, 1, A, A, None, A, 1 << 20, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 4, 4, 4, 0, 8, A, A, None, None, 0, None) == qsync.ERR_WORKSPACE
    assert f(A, 0, 4, 4, 4, 0, 8, A, A, None, A, 16, None) == qsync.ERR_WORKSPACE
    assert f(A, 0, 4, 4, 4, 0, 8, A, A, None, U, 1 << 20, None) == qsync.ERR_ALIGN
    assert f(A, 0, 0, 4, 4, 0, 8, A, A, None, None, 0, None) == qsync.OK          # empty tensor: no-op
    assert f(A, 0, 4, 4, 4, qsync.PER_ROW, 8, A, A, None, None, 0, None) in (qsync.OK, qsync.ERR_HIP)
    assert g(A, 0, 4, 4, 4, qsync.PER_ROW, 8, A, A, None, A, None, A, 1 << 20, None) == qsync.ERR_UNSUPPORTED  # colsum needs PER_TENSOR
    assert g(A, 0, 4, 4, 4, qsync.PER_COL, 8, A, A, None, None, A, A, 1 << 20, None) == qsync.ERR_UNSUPPORTED  # so does sumsq
    assert lib.qsync_absmax_workspace_bytes(4, 4, qsync.PER_ROW) == 0
    assert lib.qsync_absmax_workspace_bytes(4, 4, qsync.PER_TENSOR) > 0
    assert lib.qsync_absmax_workspace_bytes(4, 1000, qsync.PER_COL) >= 4 * 1000


def test_quantize_validation():
    f = lib.qsync_quantize
    assert f(None, 0, 4, 8, 8, 8, 8, 0, 0, 0, 0, A, A, None, None) == qsync.ERR_NULL
    assert f(A, 0, 4, 8, 8, 8, 8, 0, 0, 0, 0, A, None, None, None) == qsync.ERR_NULL       # no output at all
    assert f(A, 0, 4, 8, 8, 8, 8, 0, 0, 0, 0, None, A, None, None) == qsync.ERR_NULL       # INT8 needs a scale
    assert f(A, 0, 4, 8, 8, 12, 8, 0, 0, 0, 0, A, A, None, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 4, 8, 8, 8, 8, 0, 5, 0, 0, A, A, None, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 4, 8, 8, 8, 8, 9, 0, 0, 0, A, A, None, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 4, 8, 7, 8, 8, 0, 0, 0, 0, A, A, None, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 4, 8, 8, 8, 16, 0, 0, 0, 0, A, A, None, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 0, 8, 8, 8, 8, 0, 0, 0, 0, A, A, None, None) == qsync.OK
    assert f(A, 0, 4, 8, 8, 16, 0, 0, 0, 0, 0, None, A, None, None) in (qsync.OK, qsync.ERR_HIP)  # FP16: no scale needed


def test_qlinear_validation():
    f = lib.qsync_qlinear_fwd
    ok_args = [8, 64, 64, 64, A, A, A, A, 0, None, A, 0, None, None, 0, None]

    def call(**kw):
        names = ["tag", "M", "N", "K", "xq", "sx", "wq", "sw", "wgran", "bias", "y", "ydt", "dump", "ws", "wsb", "st"]
        a = list(ok_args)
        for k, v in kw.items():
            a[names.index(k)] = v
        return f(*a)

    assert call(xq=None) == qsync.ERR_NULL
    assert call(sx=None) == qsync.ERR_NULL
    assert call(tag=4) == qsync.ERR_BAD_ENUM
    assert call(ydt=qsync.I32) == qsync.ERR_BAD_ENUM
    assert call(wgran=4) == qsync.ERR_BAD_ENUM
    assert call(M=-5) == qsync.ERR_BAD_SHAPE
    assert call(wgran=qsync.PER_COL) == qsync.ERR_UNSUPPORTED
    assert call(tag=16, dump=A) == qsync.ERR_UNSUPPORTED
    assert call(K=40) == qsync.ERR_ALIGN                 # int8 rows must be 16-byte multiples
    assert call(tag=16, K=12) == qsync.ERR_ALIGN
    assert call(xq=U) == qsync.ERR_ALIGN
    assert call(tag=32, K=13, xq=U) in (qsync.OK, qsync.ERR_HIP)   # fp32 path has no alignment rule
    assert call(M=0) == qsync.OK
    assert call(K=(16 << 20) + 16) == qsync.ERR_UNSUPPORTED      # operand rows longer than 16 MiB
    assert call(tag=16, K=(8 << 20) + 8) == qsync.ERR_UNSUPPORTED
    # a split-K shape needs a workspace
    assert lib.qsync_qlinear_workspace_bytes(8, 64, 576, 200704) > 0
    assert call(M=64, N=576, K=200704) == qsync.ERR_WORKSPACE
    assert call(M=64, N=576, K=200704, ws=A, wsb=1024) == qsync.ERR_WORKSPACE


def test_qlinear_fwd_amax_and_scale_from_amax_validation():
    f = lib.qsync_qlinear_fwd_amax
    #        tag M   N   K  xq sx wq sw wgran bias y ydt dump amax ws wsb st
    assert f(8, 64, 64, 64, A, A, A, A, 0, None, A, 0, None, None, None, 0, None) == qsync.ERR_NULL     # no maximum word
    assert f(8, 64, 64, 64, A, A, A, A, 0, None, A, 0, None, P(4098), None, 0, None) == qsync.ERR_ALIGN   # not 4-byte aligned
    assert f(8, 64, 64, 64, None, A, A, A, 0, None, A, 0, None, A, None, 0, None) == qsync.ERR_NULL
    assert f(4, 64, 64, 64, A, A, A, A, 0, None, A, 0, None, A, None, 0, None) == qsync.ERR_BAD_ENUM
    assert f(8, 64, 64, 40, A, A, A, A, 0, None, A, 0, None, A, None, 0, None) == qsync.ERR_ALIGN
    assert f(8, 0, 64, 64, A, A, A, A, 0, None, A, 0, None, A, None, 0, None) == qsync.OK
    assert f(8, 64, 576, 200704, A, A, A, A, 0, None, A, 0, None, A, None, 0, None) == qsync.ERR_WORKSPACE   # split K
    g = lib.qsync_scale_from_amax
    assert g(None, 8, A, A, 1, None) == qsync.ERR_NULL
    assert g(A, 8, None, A, 1, None) == qsync.ERR_NULL
    assert g(A, 8, A, None, 0, None) == qsync.ERR_NULL
    assert g(A, 1, A, A, 1, None) == qsync.ERR_UNSUPPORTED
    assert g(A, 9, A, A, 1, None) == qsync.ERR_UNSUPPORTED

    g = lib.qsync_qlinear_bwd
    base = [8, 64, 64, 64, A, A, A, A, A, A, A, 0, A, 1, A, 0, None, None, 0, None, None, A, 1 << 24, None]
    assert g(*base) in (qsync.OK, qsync.ERR_HIP)
    b = list(base); b[4] = None
    assert g(*b) == qsync.ERR_NULL                       # dX wanted but no dyq
    b = list(base); b[12] = None; b[4] = None            # dX skipped: its operands may be absent
    assert g(*b) in (qsync.OK, qsync.ERR_HIP)
    b = list(base); b[16] = A                            # db without the float gradient
    assert g(*b) == qsync.ERR_NULL
    b = list(base); b[2] = 72                            # N not a multiple of 16 for the dX contraction
    assert g(*b) == qsync.ERR_ALIGN
    b = list(base); b[11] = qsync.PER_COL
    assert g(*b) == qsync.ERR_UNSUPPORTED
    b = list(base); b[13] = 9
    assert g(*b) == qsync.ERR_BAD_ENUM


def test_dequantize_validation():
    f = lib.qsync_dequantize
    assert f(None, 3, 4, 4, 4, None, None, 1.0, None, None, A, 0, None) == qsync.ERR_NULL
    assert f(A, 0, 4, 4, 4, None, None, 1.0, None, None, A, 0, None) == qsync.ERR_BAD_ENUM     # float input
    assert f(A, 3, 4, 4, 4, None, None, 1.0, None, None, A, 2, None) == qsync.ERR_BAD_ENUM     # int output
    assert f(A, 3, 4, 4, 2, None, None, 1.0, None, None, A, 0, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 3, 4, 0, 0, None, None, 1.0, None, None, A, 0, None) == qsync.OK


def test_im2col_validation():
    f = lib.qsync_im2col3x3_i8
    assert f(None, 1, 4, 4, 16, A, None, None) == qsync.ERR_NULL
    assert f(A, 1, 4, 4, 16, None, None, None) == qsync.ERR_NULL
    assert f(A, -1, 4, 4, 16, A, None, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 1, 4, 4, 24, A, None, None) == qsync.ERR_UNSUPPORTED          # C % 16
    assert f(A, 1, 3, 3, 16, None, A, None) == qsync.ERR_ALIGN                # M % 16 for the transposed copy
    assert f(U, 1, 4, 4, 16, A, None, None) == qsync.ERR_ALIGN
    assert f(A, 0, 4, 4, 16, A, None, None) == qsync.OK


def test_prepare_weights_validation():
    f = lib.qsync_prepare_weights
    ok = [A, qsync.F32, 64, 64, 8, A, A, None, A, A, A, A, A, 1 << 24, None]
    assert f(*ok) in (qsync.OK, qsync.ERR_HIP)
    for i in (0, 5, 6, 8, 9, 10, 11):
        a = list(ok); a[i] = None
        assert f(*a) == qsync.ERR_NULL
    a = list(ok); a[1] = qsync.I8
    assert f(*a) == qsync.ERR_BAD_ENUM
    a = list(ok); a[2] = -1
    assert f(*a) == qsync.ERR_BAD_SHAPE
    a = list(ok); a[4] = 9
    assert f(*a) == qsync.ERR_UNSUPPORTED
    a = list(ok); a[13] = 16
    assert f(*a) == qsync.ERR_WORKSPACE
    a = list(ok); a[12] = U
    assert f(*a) == qsync.ERR_ALIGN
    a = list(ok); a[2] = 0
    assert f(*a) == qsync.OK


def test_conv_wgrad_validation():
    f = lib.qsync_conv3x3_wgrad
    B = P(8192)                                              # 256-byte aligned
    ok = [8, 1, 4, 4, 16, 16, A, A, A, A, A, 0, None, B, 1 << 24, None]
    assert f(*ok) in (qsync.OK, qsync.ERR_HIP)
    for i in (6, 7, 8, 9, 10):
        a = list(ok); a[i] = None
        assert f(*a) == qsync.ERR_NULL
    a = list(ok); a[0] = 16; a[7] = None; a[9] = None        # binary16: no scales needed
    assert f(*a) in (qsync.OK, qsync.ERR_HIP)
    a = list(ok); a[0] = 32
    assert f(*a) == qsync.ERR_UNSUPPORTED
    a = list(ok); a[0] = 3
    assert f(*a) == qsync.ERR_BAD_ENUM
    a = list(ok); a[11] = qsync.I8
    assert f(*a) == qsync.ERR_BAD_ENUM
    a = list(ok); a[3] = 2000
    assert f(*a) == qsync.ERR_BAD_SHAPE                      # W beyond the displaced-row limit
    a = list(ok); a[0] = 16; a[3] = 600
    assert f(*a) == qsync.ERR_BAD_SHAPE                      # half that limit for two-byte elements
    a = list(ok); a[4] = 24
    assert f(*a) == qsync.ERR_ALIGN
    a = list(ok); a[5] = 8
    assert f(*a) == qsync.ERR_ALIGN
    a = list(ok); a[0] = 16; a[12] = A
    assert f(*a) == qsync.ERR_UNSUPPORTED                    # accumulator dump: INT8 only
    for nimg in (64, 63):                                    # (a contraction long enough to be split, see below)
        a = list(ok); a[1:6] = [nimg, 56, 56, 64, 64]; a[14] = 64
        assert f(*a) == qsync.ERR_WORKSPACE
        a = list(ok); a[1:6] = [nimg, 56, 56, 64, 64]; a[13] = P(4112)      # 16-byte but not 256-byte aligned
        assert f(*a) == qsync.ERR_ALIGN
    a = list(ok); a[1] = 0
    assert f(*a) == qsync.OK
    # the GEMM gathers its operands itself at any pixel count (64 images of 56 x 56 are a multiple of 128 pixels, 63 are
    # not): the workspace holds split-K partials only
    for nimg in (64, 63):
        for tag in (8, 16):
            gather = lib.qsync_conv3x3_wgrad_workspace_bytes(tag, nimg, 56, 56, 64, 64)
            assert 0 < gather < 3 * 64 * 64 * 57 * 64 // 2 and gather % (64 * 576 * 4) == 0
    assert lib.qsync_conv3x3_wgrad_workspace_bytes(8, 1, 1, 1, 16, 1 << 12) == 0          # one K tile: nothing to split
    a = list(ok); a[1:6] = [1, 1, 1, 16, 1 << 12]; a[13], a[14] = None, 0
    assert f(*a) == qsync.ERR_HIP                                                         # and none is asked for
    # from 2^24 output channels on: padded transposed copies (three of the activation, one of the gradient, 48 pixels each)
    for tag in (8, 16):
        assert lib.qsync_conv3x3_wgrad_workspace_bytes(tag, 1, 1, 1, 16, 1 << 24) >= tag // 8 * 48 * (48 + (1 << 24))
        assert lib.qsync_conv3x3_wgrad_workspace_bytes(tag, 1, 1, 1, 16, (1 << 24) - 16) < 1 << 24


@pytest.mark.parametrize("rowmajor", [False, True])
def test_gradients_share_no_launch_when_dw_lands_on_what_dx_reads(rowmajor):
    """The weight gradient may be stored over an operand of the data gradient (transposed weights, their scales, dY): in
    two launches the data gradient has read it by then.  Choice only, before any launch: fake addresses."""
    M, N, K, MB = 1024, 512, 256, 1 << 20
    at = lambda mb, off=0: (mb << 20) + off
    base = dict(dyq=at(16), dyqT=at(32), xqT=at(48), wqbT=at(64), swb=at(80), sdy=at(96), sx=at(112), dx=at(128), dw=at(144),
                acc_dw=None)

    def pair(**kw):
        b = {k: P(v) if v else None for k, v in {**base, **kw}.items()}
        if rowmajor:
            rc = lib.qsync_qlinear_bwd_rm(8, M, N, K, b["dyq"], b["sdy"], b["xqT"], b["sx"], b["wqbT"], b["swb"], qsync.PER_ROW, b["dx"],
                                          qsync.F32, b["dw"], qsync.F16, None, None, 0, None, b["acc_dw"], P(at(512)), 256 * MB, None)
        else:
            rc = lib.qsync_qlinear_bwd(8, M, N, K, b["dyq"], b["dyqT"], b["sdy"], b["xqT"], b["sx"], b["wqbT"], b["swb"], qsync.PER_ROW,
                                       b["dx"], qsync.F32, b["dw"], qsync.F16, None, None, 0, None, b["acc_dw"], P(at(512)), 256 * MB, None)
        assert rc == qsync.ERR_HIP                                # (no GPU here; the arguments themselves are fine)
        return lib.qsync_debug_last_gradient_pair()

    tile, out = pair(), 2 * N * K
    assert tile >= 0
    assert pair(wqbT=at(144)) == -1
    assert pair(wqbT=at(144, out - 16)) == -1 and pair(wqbT=at(144, out)) == tile
    assert pair(wqbT=at(144, -N * K + 16)) == -1 and pair(wqbT=at(144, -N * K)) == tile
    assert pair(dyq=at(144, out - 16)) == -1 and pair(dyq=at(144, out)) == tile
    assert pair(swb=at(144, out - 4)) == -1 and pair(sdy=at(144, 4)) == -1
    assert pair(acc_dw=at(64, -4 * N * K + 16)) == -1 and pair(acc_dw=at(64, -4 * N * K)) == tile


def test_conv_prepare_weights_validation():
    f = lib.qsync_conv3x3_prepare_weights
    ok = [A, qsync.F32, 8, 16, 8, A, A, A, A, A, A, A, 1 << 24, None]
    assert f(*ok) in (qsync.OK, qsync.ERR_HIP)
    for i in (0, 5, 6, 7, 8, 9, 10):
        a = list(ok); a[i] = None
        assert f(*a) == qsync.ERR_NULL
    a = list(ok); a[1] = qsync.I32
    assert f(*a) == qsync.ERR_BAD_ENUM
    a = list(ok); a[3] = -2
    assert f(*a) == qsync.ERR_BAD_SHAPE
    a = list(ok); a[4] = 1
    assert f(*a) == qsync.ERR_UNSUPPORTED
    a = list(ok); a[12] = 8
    assert f(*a) == qsync.ERR_WORKSPACE
    a = list(ok); a[11] = U
    assert f(*a) == qsync.ERR_ALIGN
    a = list(ok); a[2] = 0
    assert f(*a) == qsync.OK
    assert lib.qsync_conv3x3_prepare_weights_workspace_bytes(64, 64) >= 9 * 64 * 64


def test_probe_validation():
    f = lib.qsync_probe_mfma
    assert f(8, 0, 10, None, None, None) == qsync.ERR_NULL
    assert f(32, 0, 10, A, None, None) == qsync.ERR_BAD_ENUM
    assert f(8, 0, 0, A, None, None) == qsync.ERR_BAD_SHAPE
    ops = ctypes.c_double(0.0)
    assert f(16, 1, 10, A, ctypes.byref(ops), None) in (qsync.OK, qsync.ERR_HIP)
    assert ops.value == 512 * 16 * 12 * 32768.0          # iterations rounded up to a multiple of four
    assert f(16, 3, 10, A, None, None) == qsync.ERR_BAD_ENUM


def test_conv_validation():
    f = lib.qsync_conv3x3_fwd
    ok = [8, 1, 4, 4, 16, 8, A, A, A, A, qsync.PER_ROW, None, A, 0, None, None]
    names = ["tag", "nimg", "H", "W", "C", "N", "xq", "sx", "wq", "sw", "wgran", "bias", "y", "ydt", "dump", "st"]

    def call(**kw):
        a = list(ok)
        for k, v in kw.items():
            a[names.index(k)] = v
        return f(*a)

    assert call(xq=None) == qsync.ERR_NULL
    assert call(sw=None) == qsync.ERR_NULL
    assert call(tag=5) == qsync.ERR_BAD_ENUM
    assert call(ydt=qsync.I8) == qsync.ERR_BAD_ENUM
    assert call(H=-1) == qsync.ERR_BAD_SHAPE
    assert call(W=70000) == qsync.ERR_BAD_SHAPE
    assert call(nimg=1 << 20, H=64, W=64, C=64) == qsync.ERR_BAD_SHAPE        # activation beyond 2^31 bytes
    assert call(tag=32) == qsync.ERR_UNSUPPORTED
    assert call(wgran=qsync.PER_COL) == qsync.ERR_UNSUPPORTED
    assert call(tag=16, dump=A) == qsync.ERR_UNSUPPORTED
    assert call(C=24) == qsync.ERR_ALIGN
    assert call(tag=16, C=12) == qsync.ERR_ALIGN
    assert call(xq=U) == qsync.ERR_ALIGN
    assert call(nimg=0) == qsync.OK
    g = lib.qsync_conv3x3_wflip
    assert g(None, qsync.I8, 4, 4, A, None) == qsync.ERR_NULL
    assert g(A, qsync.F32, 4, 4, P(8192), None) == qsync.ERR_BAD_ENUM
    assert g(A, qsync.I8, -1, 4, P(8192), None) == qsync.ERR_BAD_SHAPE
    assert g(A, qsync.I8, 4, 4, A, None) == qsync.ERR_UNSUPPORTED             # in place
    assert g(A, qsync.I8, 0, 4, P(8192), None) == qsync.OK
    lib.qsync_debug_set_gemm_tile(1)
    lib.qsync_debug_set_gemm_tile(-1)


def test_no_gpu_gives_hip_error_not_a_crash():
    import torch
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    rc = lib.qsync_dequantize(A, 3, 4, 4, 4, None, None, 1.0, None, None, A, 0, None)
    assert rc == qsync.ERR_HIP and lib.qsync_last_hip_error() != 0


def test_absmax_quantize_validation():
    f = lib.qsync_absmax_quantize
    #        x xdt rows cols bits rnd seed off scale inv amax q qT ws wsb polls stream
    need = lib.qsync_absmax_quantize_workspace_bytes(64, 128)
    assert need == lib.qsync_absmax_workspace_bytes(64, 128, qsync.PER_TENSOR) and need > 0
    assert f(None, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, None, A, need, -1, None) == qsync.ERR_NULL
    assert f(A, 0, 64, 128, 8, 0, 0, 0, None, A, None, A, None, A, need, -1, None) == qsync.ERR_NULL
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, None, None, A, need, -1, None) == qsync.ERR_NULL      # no output
    assert f(A, 7, 64, 128, 8, 0, 0, 0, A, A, None, A, None, A, need, -1, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 64, 128, 8, 5, 0, 0, A, A, None, A, None, A, need, -1, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, -1, 128, 8, 0, 0, 0, A, A, None, A, None, A, need, -1, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 64, 128, 9, 0, 0, 0, A, A, None, A, None, A, need, -1, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 0, 128, 8, 0, 0, 0, A, A, None, A, None, None, 0, -1, None) == qsync.OK
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, None, None, 0, -1, None) == qsync.ERR_WORKSPACE
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, None, A, need - 1, -1, None) == qsync.ERR_WORKSPACE
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, None, U, need, -1, None) == qsync.ERR_ALIGN


def test_gradient_quantize_validation():
    f = lib.qsync_gradient_quantize
    #        dy dt rows cols bits rnd seed off scale inv amax colsum q qT ws wsb stream
    need = lib.qsync_absmax_workspace_bytes(64, 128, qsync.PER_TENSOR)
    assert f(None, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, A, None, A, need, None) == qsync.ERR_NULL
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, None, A, None, A, need, None) == qsync.ERR_NULL       # no column sums
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, None, None, A, need, None) == qsync.ERR_NULL       # no codes
    assert f(A, 7, 64, 128, 8, 0, 0, 0, A, A, None, A, A, None, A, need, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 64, 128, 8, 5, 0, 0, A, A, None, A, A, None, A, need, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 64, -1, 8, 0, 0, 0, A, A, None, A, A, None, A, need, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 64, 128, 1, 0, 0, 0, A, A, None, A, A, None, A, need, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 64, (1 << 19) + 8, 8, 0, 0, 0, A, A, None, A, A, None, A, need, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 0, 128, 8, 0, 0, 0, A, A, None, A, A, None, None, 0, None) == qsync.OK
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, A, None, A, need - 1, None) == qsync.ERR_WORKSPACE
    assert f(A, 0, 64, 128, 8, 0, 0, 0, A, A, None, A, A, None, U, need, None) == qsync.ERR_ALIGN


def test_convert_operands_validation():
    f = lib.qsync_convert_operands
    need = lib.qsync_absmax_workspace_bytes(64, 128, qsync.PER_TENSOR)

    def call(tag=8, x=A, xdt=0, M=64, C=128, w=A, wdt=0, N=64, taps=1, bits=8, gran=qsync.PER_ROW, sx=A, xq=A, xqT=None, wq=A, ws=A,
             wsb=need, amax=None):
        return f(tag, x, xdt, M, C, amax, w, wdt, N, taps, bits, gran, sx, A, A, xq, xqT, A, A, A, wq, A, A, A, ws, wsb, ws, wsb, None)

    assert call(tag=9) == qsync.ERR_BAD_ENUM and call(gran=qsync.PER_COL) == qsync.ERR_BAD_ENUM and call(xdt=5) == qsync.ERR_BAD_ENUM
    assert call(taps=3) == qsync.ERR_UNSUPPORTED and call(taps=9, tag=32) == qsync.ERR_UNSUPPORTED
    assert call(taps=9, xqT=A) == qsync.ERR_UNSUPPORTED and call(bits=9) == qsync.ERR_UNSUPPORTED
    assert call(x=None) == qsync.ERR_NULL and call(sx=None) == qsync.ERR_NULL and call(xq=None) == qsync.ERR_NULL
    assert call(M=-1) == qsync.ERR_BAD_SHAPE
    assert call(ws=None) == qsync.ERR_WORKSPACE and call(wsb=need - 256) == qsync.ERR_WORKSPACE and call(ws=U) == qsync.ERR_ALIGN
    assert call(M=0, w=None) == qsync.ERR_NULL            # an empty activation is no work; its weights are checked next
    assert call(M=0, N=0) == qsync.OK and call(tag=16, xq=None, N=0) == qsync.OK


def test_qlinear_backward_validation():
    f = lib.qsync_qlinear_backward
    need = lib.qsync_qlinear_bwd_workspace_bytes(16, 64, 64, 64)

    def call(tag=16, dy=A, dydt=1, dyq=None, dyqT=A, x=A, rm=0, wT=A, dx=A, dxdt=0, dw=A, db=A, ws=A, wsb=need, M=64):
        return f(tag, M, 64, 64, dy, dydt, dyq, dyqT, x, rm, wT, dx, dxdt, dw, 0, db, ws, wsb, None)

    assert call(tag=8) == qsync.ERR_UNSUPPORTED and call(tag=9) == qsync.ERR_BAD_ENUM and call(rm=2) == qsync.ERR_BAD_ENUM
    assert call(dydt=2) == qsync.ERR_BAD_ENUM and call(dxdt=2, dyqT=None, dw=None) == qsync.ERR_BAD_ENUM
    assert call(dydt=0) == qsync.ERR_UNSUPPORTED                            # fp32 is no FP16 operand as it is
    assert call(dy=None) == qsync.ERR_NULL and call(wT=None, dyqT=None, dw=None) == qsync.ERR_NULL
    assert call(dyqT=None) == qsync.ERR_NULL                                # dW reads the transposed gradient
    assert call(dyqT=None, dw=None, wsb=need - 256 if need else 0, ws=None) == qsync.ERR_WORKSPACE
    assert call(M=0, dy=A, dyqT=None, dw=None, dx=None, db=None, ws=None, wsb=0) == qsync.OK


# ---- qsync_variance_increment: a host function, so it is exercised in full here (no GPU needed) ----
class _Stats:
    def __init__(self, sumsq, amax, D):
        self.sumsq, self.amax, self.D = sumsq, amax, D


def test_variance_increment_hand_computed_cases():
    """The library's indicator on the cases worked out by hand from Prop. 3's two case equations (Indicator
    section): small integers, distinct values for every tensor, so that a swapped tensor, a dropped factor or a
    mixed-up branch changes the result.  Independent of the oracle: the expected numbers are typed in here."""
    x, v, g = _Stats(2.0, 1.0, 3), _Stats(5.0, 2.5, 7), _Stats(11.0, 0.3, 7)       # exponents 0, 1, -2
    r = qsync.qsync_variance_increment(qsync.QUANT_FIXED, x, v, g, 0.5, 0.25, 3, 2.0, 3, 10)
    s_fp = (2.0 * 0.0625 * 7 + 5.0 * 0.25 * 3) / 6
    s_bp = (11.0 * 0.0625 * 7 + 5.0 * (2.0 ** -4) * (2.0 ** -6) * 7) / 6
    assert r["sigma_fp"] == pytest.approx(s_fp, rel=1e-14) and r["sigma_bp"] == pytest.approx(s_bp, rel=1e-14)
    assert r["omega"] == pytest.approx(4.0 * 3 * s_fp + 7 * s_bp, rel=1e-14)
    r = qsync.qsync_variance_increment(qsync.QUANT_FLOAT, x, v, g, 0.0, 0.0, 3, 1.0, 2, 5)
    s_fp = (2.0 ** -6) * (2.0 * 4.0 * 7 + 5.0 * 1.0 * 3) / 6
    s_bp = (2.0 ** -6) * (11.0 * 4.0 * 7 + 5.0 * (2.0 ** -4) * 7) / 6
    assert r["sigma_fp"] == pytest.approx(s_fp, rel=1e-14) and r["sigma_bp"] == pytest.approx(s_bp, rel=1e-14)
    assert r["omega"] == pytest.approx(2 * s_fp + 3 * s_bp, rel=1e-14)


def test_variance_increment_matches_the_oracle_on_random_statistics():
    import numpy as np
    from oracle import qsync_oracle as orc
    rng = np.random.default_rng(8)
    for _ in range(200):
        st = []
        for _t in range(3):
            amax = float(np.exp(rng.uniform(-12, 6)))
            st.append(dict(sumsq=float(rng.uniform(0.1, 1e4)), amax=amax, e=orc.effective_exponent(amax),
                           D=int(rng.integers(1, 1 << 24))))
        st[int(rng.integers(0, 3))]["amax"] = float(2.0 ** int(rng.integers(-8, 8)))     # exact powers of two too
        for t in st:
            t["e"] = orc.effective_exponent(t["amax"])
        q_x, q_v = float(rng.uniform(1e-4, 1e-1)), float(rng.uniform(1e-4, 1e-1))
        k, gamma = int(rng.integers(2, 12)), float(rng.uniform(0.5, 2.0))
        d_o = int(rng.integers(0, 20)); d_L = d_o + int(rng.integers(0, 30))
        for kind, name in ((qsync.QUANT_FIXED, "fixed"), (qsync.QUANT_FLOAT, "float")):
            got = qsync.qsync_variance_increment(kind, *[_Stats(t["sumsq"], t["amax"], t["D"]) for t in st], q_x, q_v, k,
                                                 gamma, d_o, d_L)
            want = orc.variance_increment(name, *st, q_x=q_x, q_v=q_v, eps=2.0 ** -k, gamma=gamma, d_o=d_o, d_L=d_L)
            for key in ("sigma_fp", "sigma_bp", "omega"):
                assert got[key] == pytest.approx(want[key], rel=1e-12), (name, key)
    # an all-zero tensor sits in the smallest normal binade of binary32 on both sides
    z = dict(sumsq=0.0, amax=0.0, e=-126, D=16)
    one = dict(sumsq=3.0, amax=1.5, e=0, D=16)
    got = qsync.qsync_variance_increment(qsync.QUANT_FLOAT, _Stats(3.0, 1.5, 16), _Stats(0.0, 0.0, 16), _Stats(3.0, 1.5, 16),
                                         0, 0, 9, 1.0, 1, 2)
    want = orc.variance_increment("float", one, z, one, eps=2.0 ** -9, d_o=1, d_L=2)
    assert got["omega"] == pytest.approx(want["omega"], rel=1e-12)


def test_variance_increment_validation():
    f = lib.qsync_variance_increment
    S = qsync.TensorStatsC
    ok = S(1.0, 1.0, 4)
    out = ctypes.c_double()
    call = lambda kind, a, b, c, qx, qv, k, gamma, do, dl, o=out: f(kind, ctypes.byref(a) if a is not None else None,
                                                                    ctypes.byref(b) if b is not None else None,
                                                                    ctypes.byref(c) if c is not None else None, qx, qv, k, gamma, do,
                                                                    dl, None, None, ctypes.byref(o) if o is not None else None)
    assert call(0, ok, ok, ok, 0.1, 0.1, 9, 1.0, 1, 2) == qsync.OK
    assert call(0, None, ok, ok, 0.1, 0.1, 9, 1.0, 1, 2) == qsync.ERR_NULL
    assert call(0, ok, ok, ok, 0.1, 0.1, 9, 1.0, 1, 2, None) == qsync.ERR_NULL
    assert call(2, ok, ok, ok, 0.1, 0.1, 9, 1.0, 1, 2) == qsync.ERR_BAD_ENUM
    assert call(0, S(-1.0, 1.0, 4), ok, ok, 0.1, 0.1, 9, 1.0, 1, 2) == qsync.ERR_BAD_SHAPE
    assert call(0, ok, S(1.0, float("inf"), 4), ok, 0.1, 0.1, 9, 1.0, 1, 2) == qsync.ERR_BAD_SHAPE
    assert call(0, ok, ok, S(1.0, 1.0, -4), 0.1, 0.1, 9, 1.0, 1, 2) == qsync.ERR_BAD_SHAPE
    assert call(0, ok, ok, ok, 0.1, 0.1, 9, 1.0, 3, 2) == qsync.ERR_BAD_SHAPE
    assert call(0, ok, ok, ok, 0.1, 0.1, 0, 1.0, 1, 2) == qsync.ERR_UNSUPPORTED
    assert call(0, ok, ok, ok, -0.1, 0.1, 9, 1.0, 1, 2) == qsync.ERR_UNSUPPORTED
    assert call(1, ok, ok, ok, -0.1, 0.1, 9, 1.0, 1, 2) == qsync.OK            # the scales are ignored for the float kind


def test_backward_with_an_empty_batch_needs_no_workspace():
    """M = 0 with a bias gradient requested: no column-sum workspace is touched (the call clears db with a small
    kernel); without a GPU the launch itself fails, the argument check must not."""
    rc = lib.qsync_qlinear_bwd(qsync.INT8, 0, 64, 32, None, None, None, None, None, None, None, 0, None, 0, None, 0, A, A, 0,
                               None, None, None, 0, None)
    assert rc in (qsync.OK, qsync.ERR_HIP)


def test_static_scratch_absmax_validation():
    f = lib.qsync_absmax_scale_static
    assert f(None, 0, 4, 4, 4, 8, A, A, None, None, None, None) == qsync.ERR_NULL
    assert f(A, 0, 4, 4, 4, 8, None, A, None, None, None, None) == qsync.ERR_NULL
    assert f(A, qsync.I8, 4, 4, 4, 8, A, A, None, None, None, None) == qsync.ERR_BAD_ENUM
    assert f(A, 0, 4, 4, 3, 8, A, A, None, None, None, None) == qsync.ERR_BAD_SHAPE
    assert f(A, 0, 4, 4, 4, 1, A, A, None, None, None, None) == qsync.ERR_UNSUPPORTED
    assert f(A, 0, 4, 4097, 4097, 8, A, A, None, A, None, None) == qsync.ERR_WORKSPACE      # column sums beyond the scratch
    assert f(A, 0, 0, 4097, 4097, 8, A, A, None, None, None, None) == qsync.OK              # empty: no-op


def test_fp16_backward_of_int8_forward_validation():
    f = lib.qsync_qlinear_bwd_fp16_of_int8
    need = lib.qsync_qlinear_bwd_fp16_of_int8_workspace_bytes(64, 32, 48, qsync.F32)
    assert need >= 2 * (48 * 64 + 2 * 32 * 48 + 2 * 64 * 32)
    assert lib.qsync_qlinear_bwd_fp16_of_int8_workspace_bytes(64, 32, 48, qsync.F16) < need      # binary16 dY is used in place
    assert lib.qsync_qlinear_bwd_fp16_of_int8_workspace_bytes(64, 32, 48, qsync.I8) == 0
    W = P(1 << 20)                                     # 256-byte aligned fake workspace
    ok = (64, 32, 48, A, qsync.F32, A, 0, A, A, A, qsync.PER_ROW, A, qsync.F16, A, qsync.F32, A, W, need, None, None)
    chg = lambda **kw: tuple(kw.get(i, v) for i, v in zip("M N K dy dydt xqT xrm sx wq sw wgran dx dxdt dw dwdt db ws wsb offs st".split(), ok))
    assert f(*chg(xrm=2)) == qsync.ERR_BAD_ENUM
    assert f(*chg(xrm=1)) == qsync.ERR_ALIGN           # row-major activation codes: whole tiles of 128 contraction rows
    assert f(*chg(xrm=1, M=128, wsb=1 << 20)) in (qsync.OK, qsync.ERR_HIP)
    assert f(*chg(dy=None)) == qsync.ERR_NULL
    assert f(*chg(wq=None)) == qsync.ERR_NULL
    assert f(*chg(sx=None)) == qsync.ERR_NULL
    assert f(*chg(dydt=qsync.I8)) == qsync.ERR_BAD_ENUM
    assert f(*chg(wgran=qsync.PER_COL)) == qsync.ERR_BAD_ENUM
    assert f(*chg(M=-1)) == qsync.ERR_BAD_SHAPE
    assert f(*chg(N=36)) == qsync.ERR_ALIGN            # dX contracts over N: multiple of 8
    assert f(*chg(M=60)) == qsync.ERR_ALIGN            # dW contracts over M
    assert f(*chg(dy=U)) == qsync.ERR_ALIGN
    assert f(*chg(wsb=need - 1)) == qsync.ERR_WORKSPACE
    assert f(*chg(ws=None)) == qsync.ERR_WORKSPACE
    assert f(*chg(ws=P((1 << 20) + 16))) == qsync.ERR_ALIGN
    offs = (ctypes.c_size_t * 5)()
    assert f(*chg(offs=offs)) in (qsync.OK, qsync.ERR_HIP)          # valid call: only the launch can fail without a GPU
    assert list(offs) == sorted(offs) and offs[0] == 0 and all(o % 256 == 0 for o in offs)


def test_workspace_sizes_reflect_the_plans_of_the_benchmarked_shapes():
    """The workspace a backward asks for is the sum of its split-K partial sums (plus column-sum partials), so it
    shows which plan the GEMM planner picked.  Config 5's weight gradients (4096 x 1024 outputs, 16384 rows
    contracted) take four K splits of the 256x256 tile and its data gradients none; the BERT-base shapes at 8192
    tokens split their 768 x 3072 weight gradients into at most four."""
    mib = 1 << 20
    for (M, N, K) in ((16384, 4096, 1024), (16384, 1024, 4096)):
        for tag in (qsync.INT8, qsync.FP16):
            need = lib.qsync_qlinear_bwd_rm_workspace_bytes(tag, M, N, K)
            assert 4 * 16 * mib <= need < 5 * 16 * mib, (tag, M, N, K, need)
    small = lib.qsync_qlinear_bwd_rm_workspace_bytes(qsync.INT8, 8192, 3072, 768)
    assert 2 * 9 * mib <= small <= 4 * 9 * mib + 4 * mib, small


def test_row_major_backward_validation():
    f = lib.qsync_qlinear_bwd_rm
    need = lib.qsync_qlinear_bwd_rm_workspace_bytes(qsync.INT8, 256, 32, 48)
    assert need >= lib.qsync_qlinear_bwd_workspace_bytes(qsync.INT8, 256, 32, 48)
    assert lib.qsync_qlinear_bwd_rm_workspace_bytes(qsync.INT8, -1, 32, 48) == 0
    assert lib.qsync_qlinear_bwd_rm_workspace_bytes(qsync.FP32, 256, 32, 48) == 0
    W = P(1 << 20)
    ok = (qsync.INT8, 256, 32, 48, A, A, A, A, A, A, qsync.PER_ROW, A, qsync.F16, A, qsync.F32, None, None, qsync.F32, None, None, W, 1 << 20, None)
    names = "tag M N K dyq sdy xq sx wqbT swb wbgran dx dxdt dw dwdt db dyf dydt accdx accdw ws wsb st".split()
    chg = lambda **kw: tuple(kw.get(i, v) for i, v in zip(names, ok))
    assert f(*chg(dyq=None)) == qsync.ERR_NULL
    assert f(*chg(xq=None)) == qsync.ERR_NULL
    assert f(*chg(xq=None, dw=None)) in (qsync.OK, qsync.ERR_HIP)       # the activation codes serve the weight gradient only
    assert f(*chg(wqbT=None)) == qsync.ERR_NULL
    assert f(*chg(db=A)) == qsync.ERR_NULL                             # the bias gradient sums the float gradient
    assert f(*chg(dxdt=qsync.I8)) == qsync.ERR_BAD_ENUM
    assert f(*chg(wbgran=qsync.PER_COL)) == qsync.ERR_UNSUPPORTED
    assert f(*chg(M=-1)) == qsync.ERR_BAD_SHAPE
    assert f(*chg(M=192)) == qsync.ERR_ALIGN                           # whole tiles of 128 contraction rows
    assert f(*chg(N=24)) == qsync.ERR_ALIGN
    assert f(*chg(K=40)) == qsync.ERR_ALIGN
    assert f(*chg(xq=U)) == qsync.ERR_ALIGN
    assert f(*chg(M=0)) in (qsync.OK, qsync.ERR_HIP)                   # empty batch: dW is written as zeros
    assert f(*chg()) in (qsync.OK, qsync.ERR_HIP)
    assert f(*chg(tag=7)) == qsync.ERR_BAD_ENUM
    assert f(*chg(tag=qsync.FP32)) == qsync.ERR_UNSUPPORTED
    assert f(*chg(tag=qsync.FP16, N=24, sdy=None, sx=None, swb=None)) in (qsync.OK, qsync.ERR_HIP)   # binary16: multiples of 8, no scales
    assert f(*chg(tag=qsync.FP16, N=20)) == qsync.ERR_ALIGN
    assert f(*chg(tag=qsync.FP16, accdw=A)) == qsync.ERR_UNSUPPORTED
    assert f(*chg(sdy=None)) == qsync.ERR_NULL                         # INT8 needs its scales


def test_conv_forward_with_maximum_validation():
    f = lib.qsync_conv3x3_fwd_amax
    ok = [8, 1, 4, 4, 16, 16, A, A, A, A, qsync.PER_ROW, None, A, qsync.F16, None, A, None]
    assert f(*ok) in (qsync.OK, qsync.ERR_HIP)
    a = list(ok); a[15] = None
    assert f(*a) == qsync.ERR_NULL                              # the word that receives the maximum
    a = list(ok); a[15] = P(4098)
    assert f(*a) == qsync.ERR_ALIGN
    a = list(ok); a[4] = 24
    assert f(*a) == qsync.ERR_ALIGN                             # as qsync_conv3x3_fwd


def test_weight_gradient_path_of_a_convolution():
    """Which sizes the pixel ring takes: many pixels for the outputs, units enough, images it is wide enough for; every call starts from none."""
    def ring(tag, b, H, W, C, N):
        at = lambda v: P(v << 30)
        rc = lib.qsync_conv3x3_wgrad(tag, b, H, W, C, N, at(1), at(2), at(3), at(4), at(5), qsync.F32, None, at(6), 1 << 34, None)
        assert rc == qsync.ERR_HIP                                # (no GPU here; the arguments themselves are fine)
        return lib.qsync_debug_last_wgrad_ring()

    for tag, wide in ((qsync.FP16, 95), (qsync.INT8, 191)):
        assert ring(tag, 64, 56, 56, 64, 64) > 0
        assert ring(tag, 8, 14, 14, 64, 64) == 0
        assert ring(tag, 50, 20, 20, 512, 400) == 1
        assert ring(tag, 100, 16, wide, 96, 96) > 0 and ring(tag, 100, 16, wide + 1, 96, 96) == 0
    assert ring(qsync.FP16, 3, 47, 33, 424, 336) == 0             # 162 workgroups
