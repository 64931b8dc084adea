"""GPU parity: absmax/scale, quantize, cast, dequantize against the CPU oracle, element by element.

Integer codes, scales (one IEEE division each) and casts must match bit for bit; dequantized
values are held to rtol 1e-3 / atol 1e-3*max|y|.
"""
import numpy as np
import pytest
import torch

from oracle import qsync_oracle as orc
from paper_2407_02327_amd import qsync as Q
from tests.gpu_util import GRAN, RND, assert_bits_equal, assert_close, dev, empty, host, say, ws

pytestmark = pytest.mark.gpu
TORCH = {np.float32: torch.float32, np.float16: torch.float16}


def _data(rng, shape, dtype, sigma=1.0):
    x = (rng.standard_normal(shape) * sigma).astype(dtype)
    return x


def _gpu_absmax(xd, rows, cols, ld, gran, bits=8):
    n = {"tensor": 1, "row": rows, "col": cols}[gran]
    s, iv, am = empty(n, torch.float32), empty(n, torch.float32), empty(n, torch.float32)
    w = ws(Q.qsync_absmax_workspace_bytes(rows, cols, GRAN[gran]))
    Q.qsync_absmax_scale(xd, rows, cols, ld, GRAN[gran], bits, s, iv, am, None, w)
    return s, iv, am


SHAPES = [(1, 1), (3, 5), (64, 128), (130, 72), (257, 1000), (512, 4096), (1000, 24), (33, 8200)]


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("gran", ["tensor", "row", "col"])
def test_absmax_scale(dtype, gran):
    rng = np.random.default_rng(1)
    for rows, cols in SHAPES:
        for bits in (8, 4):
            say("absmax", dtype.__name__, gran, rows, cols, bits)
            x = _data(rng, (rows, cols), dtype, 3.0)
            if rows > 2:
                x[1, :] = 0                                   # an all-zero row
            s, iv, am = _gpu_absmax(dev(x), rows, cols, cols, gran, bits)
            amax = orc.absmax(x, gran)
            so, io = orc.scales_from_amax(amax, bits)
            assert_bits_equal(host(am), amax, "amax")
            assert_bits_equal(host(s), so, "scale")
            assert_bits_equal(host(iv), io, "inv_scale")


def test_absmax_strided_and_misaligned_and_zero():
    rng = np.random.default_rng(2)
    big = _data(rng, (70, 200), np.float32)
    bd = dev(big)
    for gran in ("tensor", "row", "col"):
        say("absmax strided", gran)
        view = bd[:, 3:3 + 150]                               # ld 200, base offset 12 bytes
        s, iv, am = _gpu_absmax(view, 70, 150, 200, gran)
        assert_bits_equal(host(am), orc.absmax(big[:, 3:153], gran), "amax strided")
    z = np.zeros((16, 64), np.float16)
    s, iv, am = _gpu_absmax(dev(z), 16, 64, 64, "tensor")
    assert host(s)[0] == 1 and host(iv)[0] == 1 and host(am)[0] == 0
    # large tensor: every stage-1 block is used
    say("absmax large")
    x = _data(rng, (4096, 4096), np.float16)
    x[4095, 4095] = 77.0
    s, iv, am = _gpu_absmax(dev(x), 4096, 4096, 4096, "tensor")
    assert host(am)[0] == 77.0


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_absmax_fused_with_column_sums(dtype):
    """One pass gives the per-tensor scale and the column sums (the bias gradient when x = dY)."""
    rng = np.random.default_rng(7)
    for rows, cols in [(1, 1), (3, 5), (64, 128), (257, 1000), (4096, 512), (2000, 24), (33, 8200), (16384, 64)]:
        say("absmax+colsum", dtype.__name__, rows, cols)
        x = _data(rng, (rows, cols), dtype, 1e-2)
        xd = dev(x)
        s, iv, am, cs = (empty(1, torch.float32), empty(1, torch.float32), empty(1, torch.float32),
                         empty(cols, torch.float32))
        w = ws(Q.qsync_absmax_workspace_bytes(rows, cols, Q.PER_TENSOR))
        Q.qsync_absmax_scale(xd, rows, cols, cols, Q.PER_TENSOR, 8, s, iv, am, cs, w)
        amax = orc.absmax(x, "tensor")
        so, io = orc.scales_from_amax(amax)
        assert_bits_equal(host(am), amax, "amax")
        assert_bits_equal(host(s), so, "scale")
        assert_bits_equal(host(iv), io, "inv_scale")
        assert_close(host(cs), x.astype(np.float64).sum(axis=0), "column sums")
    with pytest.raises(Q.QsyncError) as e:
        Q.qsync_absmax_scale(xd, rows, cols, cols, Q.PER_ROW, 8, s, iv, am, cs, w)
    assert e.value.status == Q.ERR_UNSUPPORTED


@pytest.mark.parametrize("k", [10, 9, 7])
def test_fp16_stochastic_cast_bit_exact(k):
    """Floating-point stochastic quantization to binary16: same draws, same integer decision, same bits."""
    rng = np.random.default_rng(31)
    for rows, cols in [(1, 1), (5, 7), (64, 64), (130, 72), (257, 1000), (1024, 768)]:
        say("fp16 SR cast", k, rows, cols)
        x = (rng.standard_normal((rows, cols)) * np.exp(rng.uniform(-14, 9, (rows, cols)))).astype(np.float32)
        if rows * cols > 16:
            x.reshape(-1)[:8] = [0.0, -0.0, 65504.0, 65530.0, 2.0 ** -24, -2.0 ** -26, 1.0, 2.0 - 2.0 ** -12]
        xd = dev(x)
        q, qt = empty((rows, cols), torch.float16), empty((cols, rows), torch.float16)
        Q.qsync_quantize(xd, rows, cols, cols, Q.FP16, k, 0, Q.ROUND_STOCHASTIC, 99, 4242, None, q, qt)
        want = orc.cast_fp16_stochastic(x, seed=99, offset=4242, k=k)
        assert_bits_equal(host(q).view(np.uint16), want.view(np.uint16), "fp16 SR")
        assert_bits_equal(host(qt).view(np.uint16), np.ascontiguousarray(want.T).view(np.uint16), "fp16 SR transposed")
    with pytest.raises(Q.QsyncError) as e:
        Q.qsync_quantize(xd, rows, cols, cols, Q.FP16, 5, 0, Q.ROUND_STOCHASTIC, 1, 0, None, q, qt)
    assert e.value.status == Q.ERR_UNSUPPORTED
    # binary16 input: a copy whatever the rounding mode
    h = x.astype(np.float16)
    Q.qsync_quantize(dev(h), rows, cols, cols, Q.FP16, 0, 0, Q.ROUND_STOCHASTIC, 1, 0, None, q, None)
    assert_bits_equal(host(q).view(np.uint16), h.view(np.uint16), "fp16 copy")


@pytest.mark.parametrize("dt", [np.float32, np.float16])
def test_prepare_weights_equals_the_separate_calls(dt):
    """Fused weight preparation (row and column maxima in one pass, both sets of codes in another) against the
    oracle's per-row and per-column quantizations; shapes on the fused path (tile edges, more row tiles than groups) and off it."""
    rng = np.random.default_rng(42)
    for (n, k) in [(64, 576), (1024, 4096), (4096, 1024), (3072, 768), (48, 40), (20, 24), (16, 8), (8208, 64), (4112, 136), (80, 264),
                   (4096, 8), (8192, 8), (8192, 16), (8192, 128)]:
        say("prepare weights", dt.__name__, n, k)
        w = (rng.standard_normal((n, k)) * 0.02).astype(dt)
        w[rng.integers(0, n), :] = 0                       # an all-zero row: scale 1
        sw, iw, aw = empty((n,), torch.float32), empty((n,), torch.float32), empty((n,), torch.float32)
        swb, iwb = empty((k,), torch.float32), empty((k,), torch.float32)
        wq, wqbT = empty((n, k), torch.int8), empty((k, n), torch.int8)
        Q.qsync_prepare_weights(dev(w), n, k, 8, sw, iw, aw, wq, swb, iwb, wqbT, ws(Q.qsync_absmax_workspace_bytes(n, k, Q.PER_COL)))
        ar, ac = orc.absmax(w, "row"), orc.absmax(w, "col")
        sr, ir = orc.scales_from_amax(ar)
        sc, ic = orc.scales_from_amax(ac)
        assert_bits_equal(host(aw), ar, "row maxima")
        assert_bits_equal(host(sw), sr, "row scales")
        assert_bits_equal(host(iw), ir, "row inverse scales")
        assert_bits_equal(host(swb), sc, "column scales")
        assert_bits_equal(host(iwb), ic, "column inverse scales")
        assert_bits_equal(host(wq), orc.quantize_int(w, ir, "row", "nearest"), "row-scaled codes")
        assert_bits_equal(host(wqbT), orc.quantize_int(w, ic, "col", "nearest").T, "column-scaled codes, transposed")


def test_im2col_on_codes_bit_exact():
    from paper_2407_02327_amd import workloads as wl
    rng = np.random.default_rng(41)
    for (b, h, w, c) in [(1, 4, 4, 16), (2, 7, 5, 16), (3, 8, 8, 64), (2, 56, 56, 64), (1, 13, 16, 48)]:
        say("im2col codes", b, h, w, c)
        xq = rng.integers(-127, 128, (b, h, w, c)).astype(np.int8)
        M, K = b * h * w, 9 * c
        want = wl.im2col_nhwc_3x3(xq)
        a = empty((M, K), torch.int8); a.fill_(5)
        aT = None
        if M % 16 == 0:
            aT = empty((K, M), torch.int8); aT.fill_(5)
        Q.qsync_im2col3x3_i8(dev(xq), b, h, w, c, a, aT)
        assert_bits_equal(host(a), want, "patch matrix")
        if aT is not None:
            assert_bits_equal(host(aT), np.ascontiguousarray(want.T), "transposed patch matrix")
            a2 = empty((K, M), torch.int8)
            Q.qsync_im2col3x3_i8(dev(xq), b, h, w, c, None, a2)            # transposed copy alone
            assert_bits_equal(host(a2), np.ascontiguousarray(want.T), "transposed patch matrix alone")


def test_absmax_workspace_is_reusable_without_clearing():
    """The arrival counters at the start of the workspace are zeroed once by the caller and left zero
    by every call: one buffer serves a sequence of different reductions, each checked against the oracle."""
    rng = np.random.default_rng(11)
    shapes = [(4096, 4096), (64, 128), (16384, 1024), (257, 1000), (8192, 72), (33, 8200), (3, 5), (4096, 4096)]
    nbytes = max(max(Q.qsync_absmax_workspace_bytes(r, c, Q.PER_TENSOR), Q.qsync_absmax_workspace_bytes(r, c, Q.PER_COL))
                 for r, c in shapes)
    w = ws(nbytes)
    for rep, (rows, cols) in enumerate(shapes):
        dtype = np.float16 if rep % 2 == 0 else np.float32
        x = _data(rng, (rows, cols), dtype, 0.5)
        xd = dev(x)
        for gran, with_sums in (("tensor", False), ("col", False), ("tensor", True)):
            say("absmax reuse", rows, cols, dtype.__name__, gran, with_sums)
            n = 1 if gran == "tensor" else cols
            sc, iv, am = empty(n, torch.float32), empty(n, torch.float32), empty(n, torch.float32)
            cs = empty(cols, torch.float32) if with_sums else None
            Q.qsync_absmax_scale(xd, rows, cols, cols, GRAN[gran], 8, sc, iv, am, cs, w)
            amax = orc.absmax(x, gran)
            so, io = orc.scales_from_amax(amax)
            assert_bits_equal(host(am), amax, "amax")
            assert_bits_equal(host(sc), so, "scale")
            assert_bits_equal(host(iv), io, "inv_scale")
            if with_sums:
                assert_close(host(cs), x.astype(np.float64).sum(axis=0), "column sums")
    assert int(w[:256].to(torch.int32).abs().sum().item()) == 0, "the arrival counter must be left at zero"


def test_absmax_column_sums_are_reproducible():
    """The in-kernel fold uses a fixed assignment and order: two runs give identical bits."""
    rng = np.random.default_rng(12)
    rows, cols = 16384, 4096
    xd = dev(_data(rng, (rows, cols), np.float16, 1e-2))
    w = ws(Q.qsync_absmax_workspace_bytes(rows, cols, Q.PER_TENSOR))
    outs = []
    for _ in range(3):
        sc, iv, am, cs = (empty(1, torch.float32), empty(1, torch.float32), empty(1, torch.float32),
                          empty(cols, torch.float32))
        Q.qsync_absmax_scale(xd, rows, cols, cols, Q.PER_TENSOR, 8, sc, iv, am, cs, w)
        outs.append((host(cs).copy(), host(sc).copy()))
    for cs, sc in outs[1:]:
        assert_bits_equal(cs, outs[0][0], "column sums, repeated run")
        assert_bits_equal(sc, outs[0][1], "scale, repeated run")


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_absmax_with_squared_norm(dtype):
    """The indicator statistics: one pass yields the scale, the squared norm and (optionally) the column sums."""
    rng = np.random.default_rng(13)
    for rows, cols in [(1, 1), (3, 5), (64, 128), (257, 1000), (4096, 512), (33, 8200), (16384, 1024)]:
        for with_sums in (False, True):
            say("absmax+sumsq", dtype.__name__, rows, cols, with_sums)
            x = _data(rng, (rows, cols), dtype, 0.7)
            xd = dev(x)
            sc, iv, am, sq = (empty(1, torch.float32) for _ in range(4))
            cs = empty(cols, torch.float32) if with_sums else None
            w = ws(Q.qsync_absmax_workspace_bytes(rows, cols, Q.PER_TENSOR))
            Q.qsync_absmax_scale(xd, rows, cols, cols, Q.PER_TENSOR, 8, sc, iv, am, cs, w, sumsq_opt=sq)
            st = orc.tensor_stats(x)
            assert_bits_equal(host(am), orc.absmax(x, "tensor"), "amax")
            assert_bits_equal(host(sc), orc.scales_from_amax(orc.absmax(x, "tensor"))[0], "scale")
            assert abs(float(host(sq)[0]) - st["sumsq"]) <= 1e-4 * st["sumsq"] + 1e-30, (float(host(sq)[0]), st["sumsq"])
            if with_sums:
                assert_close(host(cs), x.astype(np.float64).sum(axis=0), "column sums")


def test_indicator_from_device_statistics_matches_oracle():
    from paper_2407_02327_amd import indicator as ind
    rng = np.random.default_rng(14)
    w = (rng.standard_normal((768, 512)) * 0.02).astype(np.float32)
    v = rng.standard_normal((2048, 512)).astype(np.float16)
    g = (rng.standard_normal((2048, 768)) * 1e-3).astype(np.float16)
    sw, sv, sg = ind.tensor_stats(dev(w)), ind.tensor_stats(dev(v)), ind.tensor_stats(dev(g))
    ow, ov, og = orc.tensor_stats(w), orc.tensor_stats(v), orc.tensor_stats(g)
    for got, want in ((sw, ow), (sv, ov), (sg, og)):
        assert got.amax == want["amax"] and got.D == want["D"]
        assert abs(got.sumsq - want["sumsq"]) <= 1e-4 * want["sumsq"]
    q_x, q_v = ow["amax"] / 127, ov["amax"] / 127
    for kind in ("fixed", "float"):
        a = ind.variance_increment(kind, sw, sv, sg, q_x=q_x, q_v=q_v, k=9, gamma=1.5, d_o=3, d_L=24)
        b = orc.variance_increment(kind, ow, ov, og, q_x=q_x, q_v=q_v, eps=2.0 ** -9, gamma=1.5, d_o=3, d_L=24)
        for k in ("sigma_fp", "sigma_bp", "omega"):
            assert a[k] == pytest.approx(b[k], rel=2e-4), (kind, k)


def _gpu_quantize(xd, rows, cols, ld, tag, gran, rnd, seed, offset, inv, want_q=True, want_t=True, bits=8):
    dt = {Q.INT8: torch.int8, Q.FP16: torch.float16, Q.FP32: torch.float32}[tag]
    q = empty((rows, cols), dt) if want_q else None
    qt = empty((cols, rows), dt) if want_t else None
    if q is not None:
        q.fill_(3)
    if qt is not None:
        qt.fill_(3)
    Q.qsync_quantize(xd, rows, cols, ld, tag, bits, GRAN[gran], RND[rnd], seed, offset, inv, q, qt)
    return q, qt


QSHAPES = [(16, 16), (16, 8), (48, 24), (128, 128), (256, 136), (144, 1000), (1024, 768), (5, 7), (17, 40), (24, 16),
           (130, 66), (2048, 64)]


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("gran", ["tensor", "row", "col"])
@pytest.mark.parametrize("rnd", ["nearest", "stochastic", "floor"])
def test_quantize_int8(dtype, gran, rnd):
    rng = np.random.default_rng(3)
    for rows, cols in QSHAPES:
        say("quantize", dtype.__name__, gran, rnd, rows, cols)
        x = _data(rng, (rows, cols), dtype, 0.7)
        x[0, 0] = 0
        seed, offset = 0x1234_5678_9ABC_DEF0 + rows, (1 << 64) - 5 if rows == 48 else 1000 * cols
        amax = orc.absmax(x, gran)
        so, io = orc.scales_from_amax(amax)
        want = orc.quantize_int(x, io, gran, rnd, seed, offset)
        q, qt = _gpu_quantize(dev(x), rows, cols, cols, Q.INT8, gran, rnd, seed, offset, dev(io))
        assert_bits_equal(host(q), want, "codes")
        assert_bits_equal(host(qt), want.T, "transposed codes")
    # only one of the two outputs; fewer bits
    x = _data(rng, (64, 64), dtype)
    so, io = orc.scales_from_amax(orc.absmax(x, gran), 5)
    want = orc.quantize_int(x, io, gran, rnd, 9, 9, bits=5)
    q, _ = _gpu_quantize(dev(x), 64, 64, 64, Q.INT8, gran, rnd, 9, 9, dev(io), True, False, bits=5)
    _, qt = _gpu_quantize(dev(x), 64, 64, 64, Q.INT8, gran, rnd, 9, 9, dev(io), False, True, bits=5)
    assert_bits_equal(host(q), want, "codes 5 bit")
    assert_bits_equal(host(qt), want.T, "transposed codes 5 bit")
    assert np.abs(want).max() == 15


def test_quantize_strided_input_and_special_values():
    rng = np.random.default_rng(4)
    for ld in (300, 304):                                      # ld 300: rows not 16-byte multiples -> scalar path
        big = _data(rng, (96, ld), np.float16)
        x = big[:, 8:8 + 256]
        so, io = orc.scales_from_amax(orc.absmax(x))
        say("quantize strided", ld)
        q, qt = _gpu_quantize(dev(big)[:, 8:264], 96, 256, ld, Q.INT8, "tensor", "stochastic", 5, 0, dev(io))
        want = orc.quantize_int(np.ascontiguousarray(x), io, "tensor", "stochastic", 5, 0)
        assert_bits_equal(host(q), want, "strided codes")
        assert_bits_equal(host(qt), want.T, "strided transposed codes")
    # ties, +-amax, subnormal inputs, exact integers
    say("quantize special values")
    t = np.zeros((16, 16), np.float32)
    t[0, :8] = [127.0, 0.5, 1.5, 2.5, -0.5, -1.5, -2.5, 3.5]
    t[1, :4] = [-127.0, 1e-41, -1e-41, 126.5]
    so, io = orc.scales_from_amax(orc.absmax(t))
    for rnd in ("nearest", "stochastic", "floor"):
        q, qt = _gpu_quantize(dev(t), 16, 16, 16, Q.INT8, "tensor", rnd, 11, 3, dev(io))
        assert_bits_equal(host(q), orc.quantize_int(t, io, "tensor", rnd, 11, 3), f"special {rnd}")
    assert host(q).min() >= -127


@pytest.mark.parametrize("src", [np.float32, np.float16])
@pytest.mark.parametrize("tag", [Q.FP16, Q.FP32])
def test_cast_and_transpose(src, tag):
    rng = np.random.default_rng(5)
    for rows, cols in [(1, 1), (64, 64), (70, 130), (300, 96), (33, 1000), (256, 200), (72, 1032), (8, 8), (4096, 64),
                       (520, 8)]:
        say("cast", src.__name__, tag, rows, cols)
        x = _data(rng, (rows, cols), src, 100.0)
        x[0, 0] = 1.0 + 2.0**-11 if src == np.float32 else x[0, 0]     # an exact tie for binary16
        q, qt = _gpu_quantize(dev(x), rows, cols, cols, tag, "tensor", "nearest", 0, 0, None)
        want = orc.cast_fp16(x) if tag == Q.FP16 else x.astype(np.float32)
        assert_bits_equal(host(q), want, "cast")
        assert_bits_equal(host(qt), want.T, "cast transposed")
        q1, _ = _gpu_quantize(dev(x), rows, cols, cols, tag, "tensor", "nearest", 0, 0, None, True, False)
        _, qt1 = _gpu_quantize(dev(x), rows, cols, cols, tag, "tensor", "nearest", 0, 0, None, False, True)
        assert_bits_equal(host(q1), want, "cast, plain copy alone")
        assert_bits_equal(host(qt1), want.T, "cast, transposed copy alone")


@pytest.mark.parametrize("adt", [np.int32, np.int8])
@pytest.mark.parametrize("ydt", [np.float32, np.float16])
def test_dequantize(adt, ydt):
    rng = np.random.default_rng(6)
    for rows, cols in [(1, 1), (64, 64), (37, 53), (256, 1024), (100, 12)]:
        say("dequantize", adt.__name__, ydt.__name__, rows, cols)
        lim = 127 if adt == np.int8 else 2_000_000
        a = rng.integers(-lim, lim + 1, size=(rows, cols)).astype(adt)
        rs = rng.uniform(0.5, 2, rows).astype(np.float32)
        cs = rng.uniform(1e-4, 2e-4, cols).astype(np.float32)
        cb = rng.standard_normal(cols).astype(np.float32)
        for use in [(False, False, False), (True, False, False), (False, True, True), (True, True, True)]:
            y = empty((rows, cols), TORCH[ydt])
            Q.qsync_dequantize(dev(a), rows, cols, cols, dev(rs) if use[0] else None, dev(cs) if use[1] else None,
                               0.01, dev(cb) if use[2] else None, y)
            want = orc.dequantize(a, 0.01, rs if use[0] else None, cs if use[1] else None, cb if use[2] else None,
                                  np.float64)
            assert_close(host(y), want, "dequantize")
    # strided input
    a = rng.integers(-1000, 1000, size=(20, 64)).astype(adt if adt == np.int32 else np.int8)
    y = empty((20, 40), TORCH[ydt])
    Q.qsync_dequantize(dev(a)[:, 4:44], 20, 40, 64, None, None, 0.5, None, y)
    assert_close(host(y), a[:, 4:44] * 0.5, "dequantize strided")


@pytest.mark.parametrize("ydt", [np.float32, np.float16])
@pytest.mark.parametrize("rows,cols", [(1, 3), (1, 4), (1, 8), (3, 5), (1, 1023), (255, 8), (257, 31), (1, (1 << 20) - 1), (1, 1 << 20), (1025, 1031), (4099, 4093),
                                       (4096, 4096)])
def test_dequantize_contiguous_codes_of_any_length(ydt, rows, cols):
    """Contiguous int8 codes with one scale, around a vector, a workgroup and the sizes where more vectors go to a thread; at addresses
    that are vectors and that are not: bits of the oracle's single rounding."""
    rng = np.random.default_rng(rows * cols)
    a = rng.integers(-127, 128, size=(rows, cols)).astype(np.int8)
    scale = np.float32(0.0123456789)
    want = orc.dequantize(a, float(scale), out_dtype=ydt)
    for off_a, off_y in ((0, 0), (1, 0), (4, 0), (0, 1)):
        say("dequantize flat", ydt.__name__, rows, cols, off_a, off_y)
        src = torch.zeros(rows * cols + off_a, dtype=torch.int8, device="cuda")
        src[off_a:] = dev(a.reshape(-1))
        y = torch.full((rows * cols + off_y + 8,), 7.0, dtype=TORCH[ydt], device="cuda")
        Q.qsync_dequantize(src[off_a:], rows, cols, cols, None, None, 1.0, None, y[off_y:], tensor_scale_dev_opt=dev(np.array([scale])))
        assert_bits_equal(host(y)[off_y:off_y + rows * cols].reshape(rows, cols), want, "dequantize")
        assert (host(y)[:off_y] == 7.0).all() and (host(y)[off_y + rows * cols:] == 7.0).all()


@pytest.mark.parametrize("ydt", [torch.float32, torch.float16])
@pytest.mark.parametrize("more", [-1, 0, 13])
def test_dequantize_outputs_around_128_MB(ydt, more):
    """The size from which outputs are streamed: bits of the same codes dequantized in pieces, which are not."""
    n = (1 << 27) // (4 if ydt == torch.float32 else 2) + more
    say("dequantize around 128 MB", ydt, more)
    a = torch.randint(-127, 128, (n,), dtype=torch.int8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(more + 5))
    scale = torch.full((1,), 0.0123456789, device="cuda")
    y, want = (torch.full((n + 8,), 7.0, dtype=ydt, device="cuda") for _ in range(2))
    Q.qsync_dequantize(a, 1, n, n, None, None, 1.0, None, y, tensor_scale_dev_opt=scale)
    for at in range(0, n, 1 << 22):
        k = min(1 << 22, n - at)
        Q.qsync_dequantize(a[at:], 1, k, k, None, None, 1.0, None, want[at:], tensor_scale_dev_opt=scale)
    assert torch.equal(y.view(torch.uint8), want.view(torch.uint8)) and (y[n:] == 7.0).all()


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("rnd", ["nearest", "stochastic", "floor"])
@pytest.mark.parametrize("rows,cols", [(1, 7), (1, 8), (1, 9), (3, 5), (5, 3), (91, 11), (1, 8191), (8193, 1), (1024, 9), (33, 999), (1, 249999), (1, 250001),
                                       (8195, 31), (389999, 1), (1, 390001), (399, 1001), (515, 777)])
def test_quantize_contiguous_rows_of_any_length(dtype, rnd, rows, cols):
    """Codes of a contiguous tensor whose rows are no multiple of eight, around a group and a workgroup's groups and the sizes from
    which groups are what a thread takes, at addresses that are vectors and that are not: bits of the oracle."""
    rng = np.random.default_rng(rows + cols)
    x = _data(rng, (rows, cols), dtype, 0.7)
    _, io = orc.scales_from_amax(orc.absmax(x, "tensor"))
    want = orc.quantize_int(x, io, "tensor", rnd, 77, (1 << 64) - 3)
    codes = {"nearest": Q.ROUND_NEAREST, "stochastic": Q.ROUND_STOCHASTIC, "floor": Q.ROUND_FLOOR}[rnd]
    for off_x, off_q in ((0, 0), (1, 0), (0, 3)):
        say("quantize flat", dtype.__name__, rnd, rows, cols, off_x, off_q)
        src = torch.zeros(rows * cols + off_x, dtype=TORCH[dtype], device="cuda")
        src[off_x:] = dev(x.reshape(-1))
        q = torch.full((rows * cols + off_q + 8,), 99, dtype=torch.int8, device="cuda")
        Q.qsync_quantize(src[off_x:], rows, cols, cols, Q.INT8, 8, Q.PER_TENSOR, codes, 77, (1 << 64) - 3, dev(io), q[off_q:], None)
        assert_bits_equal(host(q)[off_q:off_q + rows * cols].reshape(rows, cols), want, "codes")
        assert (host(q)[:off_q] == 99).all() and (host(q)[off_q + rows * cols:] == 99).all()


def test_dequantize_to_binary16_rounds_the_exact_product_once():
    """int8 codes times one binary32 scale, binary16 output: the result is the exact product rounded once, bit
    for bit, also on inputs where rounding to binary32 first would give the other neighbour."""
    rng = np.random.default_rng(3)
    n = 1 << 18
    scales = (rng.uniform(0.5, 1.0, size=n).astype(np.float32) * np.float32(2.0 ** -7))
    codes = rng.integers(-127, 128, size=n).astype(np.int8)
    twice = (codes.astype(np.float32) * scales).astype(np.float16)
    want = orc.dequantize(codes.reshape(-1, 1), 1.0, row_scale=scales, out_dtype=np.float16)
    assert (want.reshape(-1).view(np.uint16) != twice.view(np.uint16)).sum() >= 3
    say("dequantize once-rounded, per-row scales")
    y = empty((n, 1), torch.float16)
    Q.qsync_dequantize(dev(codes.reshape(-1, 1)), n, 1, 1, dev(scales), None, 1.0, None, y)
    assert_bits_equal(host(y), want, "per-row scale")
    # the same pairs with the scale along the columns (the vector kernel), and a tensor scale held on the device
    rows = 64
    a = np.tile(codes[:4096].reshape(1, -1), (rows, 1))
    want = orc.dequantize(a, 1.0, col_scale=scales[:4096], out_dtype=np.float16)
    y = empty((rows, 4096), torch.float16)
    Q.qsync_dequantize(dev(a), rows, 4096, 4096, None, dev(scales[:4096]), 1.0, None, y)
    assert_bits_equal(host(y), want, "per-column scale")
    for i in np.flatnonzero(want[0].view(np.uint16) != twice[:4096].view(np.uint16))[:3]:
        a1 = rng.integers(-127, 128, size=(48, 272)).astype(np.int8)
        a1[0, 0] = codes[i]
        y = empty(a1.shape, torch.float16)
        Q.qsync_dequantize(dev(a1), 48, 272, 272, None, None, 1.0, None, y, tensor_scale_dev_opt=dev(scales[i:i + 1]))
        assert_bits_equal(host(y), orc.dequantize(a1, float(scales[i]), out_dtype=np.float16), "tensor scale on the device")


def test_empty_tensors_are_noops():
    s = empty(1, torch.float32)
    a = empty(1, torch.int32)
    Q.qsync_absmax_scale(s, 0, 16, 16, Q.PER_TENSOR, 8, s, s, None, None, None)
    Q.qsync_quantize(s, 0, 16, 16, Q.INT8, 8, 0, 0, 0, 0, s, s, None)
    Q.qsync_dequantize(a, 16, 0, 0, None, None, 1.0, None, s)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("rnd", ["nearest", "stochastic", "floor"])
def test_absmax_quantize_in_one_launch(dtype, rnd):
    """qsync_absmax_quantize: maximum, scales, codes and transposed codes equal the oracle's absmax ->
    scales_from_amax -> quantize_int bit for bit -- on shapes the single launch serves (up to 128 KB: 64x504, for fp32
    64x512 is the last, for binary16 128x512), on shapes that take block maxima and a quantizing pass, on shapes handed to
    the two separate passes (odd columns), for any poll_limit, and on repeated calls that share one workspace without
    clearing it."""
    rng = np.random.default_rng(31)
    shapes = [(64, 128), (272, 1000), (1008, 72), (4096, 768), (2048, 2048), (48, 8200), (130, 72), (3, 5), (257, 1001),
              (64, 504), (64, 512), (64, 520), (128, 512), (128, 520)]
    w = ws(max(Q.qsync_absmax_quantize_workspace_bytes(r, c) for r, c in shapes))       # zero-filled once
    for rows, cols in shapes:
        x = _data(rng, (rows, cols), dtype, sigma=0.3)
        x[rows // 2, cols // 3] = dtype(-7.5)                                          # the maximum, negative
        xd = dev(x)
        amax = orc.absmax(x, "tensor")
        so, io = orc.scales_from_amax(amax)
        want = orc.quantize_int(x, io, "tensor", rnd, 77, 1234)
        for with_t, polls in ((True, -1), (False, 0)):
            say("absmax_quantize", dtype.__name__, rnd, rows, cols, "polls", polls, "transposed", with_t)
            s, iv, am = empty(1, torch.float32), empty(1, torch.float32), empty(1, torch.float32)
            q = torch.full((rows, cols), 99, dtype=torch.int8, device="cuda")
            qT = torch.full((cols, rows), 99, dtype=torch.int8, device="cuda") if with_t else None
            Q.qsync_absmax_quantize(xd, rows, cols, 8, RND[rnd], 77, 1234, s, iv, am, q, qT, w, polls)
            torch.cuda.synchronize()
            assert_bits_equal(host(am), amax, "amax")
            assert_bits_equal(host(s), so, "scale")
            assert_bits_equal(host(iv), io, "inverse scale")
            assert_bits_equal(host(q), want, "codes")
            if with_t:
                assert_bits_equal(host(qT), want.T, "transposed codes")
    # the workspace's arrival counter is zero: the separate maximum pass can use the same buffer next
    assert int(w[:4].view(torch.int32).item()) == 0
    x = _data(rng, (512, 4096), dtype)
    s, iv, am = empty(1, torch.float32), empty(1, torch.float32), empty(1, torch.float32)
    Q.qsync_absmax_scale(dev(x), 512, 4096, 4096, Q.PER_TENSOR, 8, s, iv, am, None, w)
    torch.cuda.synchronize()
    assert_bits_equal(host(am), orc.absmax(x, "tensor"), "amax by the separate pass on the shared workspace")


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_gradient_quantize(dtype):
    """qsync_gradient_quantize: maximum, scales and codes bit for bit those of the oracle, column sums within the bound of a
    recursive fp32 sum, (rows - 1) 2^-24 sum |x| per column: at the last sizes of the single launch (128 KB; 512 rows), on
    both tile heights and the streaming form, around the fold's sixteen columns, and on shapes handed to the two calls."""
    rng = np.random.default_rng(47)
    per = 16 // np.dtype(dtype).itemsize                            # 64 x (128 per) elements are 128 KB
    shapes = [(64, 128 * per), (64, 128 * per + 8), (512, 16), (513, 16), (128, 72), (16, 24), (1808, 1040), (272, 1000),
              (4096, 2056), (45, 1024), (500, 800), (3, 5), (257, 1001)]
    w = ws(max(Q.qsync_absmax_workspace_bytes(r, c, Q.PER_TENSOR) for r, c in shapes))
    for rows, cols in shapes:
        x = _data(rng, (rows, cols), dtype, sigma=0.3)
        x[rows // 2, cols // 3] = dtype(-7.5)
        amax = orc.absmax(x, "tensor")
        so, io = orc.scales_from_amax(amax)
        xd, x64 = dev(x), x.astype(np.float64)
        bound = (rows - 1) * 2.0 ** -24 * np.abs(x64).sum(0) + 1e-30
        for rnd, with_t in (("stochastic", True), ("nearest", False)):
            say("gradient_quantize", dtype.__name__, rnd, rows, cols, "transposed", with_t)
            want = orc.quantize_int(x, io, "tensor", rnd, 77, 1234)
            s, iv, am = (torch.full((1,), -3.0, dtype=torch.float32, device="cuda") for _ in range(3))
            cs = torch.full((cols,), -3.0, dtype=torch.float32, device="cuda")
            q = torch.full((rows, cols), 99, dtype=torch.int8, device="cuda")
            qT = torch.full((cols, rows), 99, dtype=torch.int8, device="cuda") if with_t else None
            Q.qsync_gradient_quantize(xd, rows, cols, 8, RND[rnd], 77, 1234, s, iv, am, cs, q, qT, w)
            assert_bits_equal(host(am), amax, "amax")
            assert_bits_equal(host(s), so, "scale")
            assert_bits_equal(host(iv), io, "inverse scale")
            assert_bits_equal(host(q), want, "codes")
            if with_t:
                assert_bits_equal(host(qT), want.T, "transposed codes")
            assert np.all(np.abs(host(cs).astype(np.float64) - x64.sum(0)) <= bound), "column sums"


@pytest.mark.parametrize("power", [-140, -120, -101, -100, -20, 3, 15, 99, 100, 101])
def test_stochastic_codes_for_any_inverse_scale(power):
    """Binary16 values times 2^16 times the inverse scale in one multiplication inside 2^-100 .. 2^100, in two outside:
    the oracle's codes either way, clamped, subnormal and zero products among them, streaming and tiled.  (These draws hold
    no 65535, the one draw for which a negative product below 2^-24 is floor(x inv) here and 0 in the oracle, whose
    residual rounds to 1.)"""
    say("stochastic codes, inverse scale 1.37 * 2^", power)
    rng = np.random.default_rng(12)
    x = _data(rng, (96, 264), np.float16, sigma=0.4)
    x.reshape(-1)[:6] = np.array([65504.0, -65504.0, 2.0 ** -24, -2.0 ** -24, 0.0, -0.0], np.float16)
    inv = np.array([1.37 * 2.0 ** power], np.float32)
    want = orc.quantize_int(x, inv, "tensor", "stochastic", 5, 99)
    for with_t in (False, True):
        q, qT = empty((96, 264), torch.int8), empty((264, 96), torch.int8) if with_t else None
        Q.qsync_quantize(dev(x), 96, 264, 264, Q.INT8, 8, Q.PER_TENSOR, Q.ROUND_STOCHASTIC, 5, 99, dev(inv), q, qT)
        assert_bits_equal(host(q), want, "codes")
        if with_t:
            assert_bits_equal(host(qT), want.T, "transposed codes")


OPERANDS = [
    # tag, weight granularity, taps, M, C, N, transposed activation copy: whole tensors (128 KB) on either side, around 16 rows, tiles
    # and streaming, odd row counts, shapes that no shared launch takes (odd columns; N % 16)
    ("int8", "tensor", 1, 64, 128, 128, True), ("int8", "tensor", 1, 512, 1024, 64, False), ("int8", "tensor", 1, 64, 256, 1024, True),
    ("int8", "tensor", 1, 272, 1000, 304, True), ("int8", "row", 1, 64, 128, 128, True), ("int8", "row", 1, 1808, 784, 1040, True),
    ("int8", "row", 1, 2048, 768, 768, False), ("int8", "row", 1, 45, 1024, 256, True), ("int8", "row", 1, 130, 72, 48, True),
    ("int8", "row", 1, 16, 8, 8192, False), ("int8", "row", 1, 64, 33, 16, True), ("int8", "row", 1, 64, 64, 24, True),
    ("int8", "row", 9, 3 * 7 * 9, 16, 32, False), ("int8", "row", 9, 4 * 14 * 14, 64, 48, False), ("int8", "tensor", 9, 99, 16, 16, False),
    ("fp16", "row", 1, 2056, 1032, 1000, True), ("fp16", "row", 1, 65, 72, 8, True), ("fp16", "row", 1, 64, 33, 7, True),
    ("fp16", "row", 9, 4704, 64, 40, False), ("fp16", "row", 9, 99, 8, 8, False), ("fp32", "row", 1, 260, 132, 64, True),
    ("fp32", "row", 1, 33, 7, 5, True)]


@pytest.mark.parametrize("case,x_from", [(c, x) for c in OPERANDS for x in ("float32", "float16", "amax" if c[0] == "int8" else "in place")],
                         ids=lambda c: c if isinstance(c, str) else "-".join(map(str, c)))
def test_convert_operands_equals_the_separate_calls(case, x_from):
    """qsync_convert_operands against its definition, the separate calls, bit for bit in every output; once more with one
    workspace for both operands, which has to fall back to one conversion after the other."""
    tag, gran, taps, M, C, N, with_t = case
    say("convert_operands", *case, x_from)
    i8, K = tag == "int8", taps * C
    code, qd = {"int8": (Q.INT8, torch.int8), "fp16": (Q.FP16, torch.float16), "fp32": (Q.FP32, torch.float32)}[tag]
    rng = np.random.default_rng(M + 7 * C + N)
    x = dev(_data(rng, (M, C), np.float32 if x_from == "float32" else np.float16, sigma=0.5))
    w = dev(_data(rng, (N, K), np.float32, sigma=0.02))
    ns, nsb = (N, C) if gran == "row" else (1, 1)
    need = max(Q.qsync_absmax_workspace_bytes(M, C, Q.PER_TENSOR), Q.qsync_absmax_workspace_bytes(N, K, Q.PER_TENSOR),
               Q.qsync_conv3x3_prepare_weights_workspace_bytes(N, C) if taps == 9 else 0)
    g = Q.PER_ROW if gran == "row" else Q.PER_TENSOR

    def buffers():
        f = lambda n: torch.full((n,), -3.0, dtype=torch.float32, device="cuda")
        e = lambda r, c: torch.full((r, c), 77, dtype=qd, device="cuda")
        inp = x_from == "in place"
        return dict(sx=f(1), ix=f(1), ax=f(1), sw=f(ns), iw=f(ns), aw=f(ns), swb=f(nsb), iwb=f(nsb), xq=None if inp else e(M, C),
                    xqT=e(C, M) if with_t else None, wq=e(N, K), wqbT=e(C, taps * N),
                    amax=x.float().abs().max().reshape(1).clone() if x_from == "amax" else None)

    def separate(b, wx, ww):
        if i8 and b["amax"] is None:
            Q.qsync_absmax_quantize(x, M, C, 8, Q.ROUND_NEAREST, 0, 0, b["sx"], b["ix"], b["ax"], b["xq"], b["xqT"], wx)
        elif i8:
            Q.qsync_scale_from_amax(b["amax"], 8, b["sx"], b["ix"], True)
            Q.qsync_quantize(x, M, C, C, Q.INT8, 8, Q.PER_TENSOR, Q.ROUND_NEAREST, 0, 0, b["ix"], b["xq"], b["xqT"])
        elif b["xq"] is not None or b["xqT"] is not None:
            Q.qsync_quantize(x, M, C, C, code, 0, 0, 0, 0, 0, None, b["xq"], b["xqT"])
        if i8 and gran == "row" and taps == 9:
            Q.qsync_conv3x3_prepare_weights(w, N, C, 8, b["sw"], b["iw"], b["wq"], b["swb"], b["iwb"], b["wqbT"], ww)
        elif i8 and gran == "row":
            Q.qsync_prepare_weights(w, N, C, 8, b["sw"], b["iw"], b["aw"], b["wq"], b["swb"], b["iwb"], b["wqbT"], ww)
        else:
            wT = b["wqbT"] if taps == 1 else None
            if i8:
                Q.qsync_absmax_quantize(w, N, K, 8, Q.ROUND_NEAREST, 0, 0, b["sw"], b["iw"], b["aw"], b["wq"], wT, ww)
            else:
                Q.qsync_quantize(w, N, K, K, code, 0, 0, 0, 0, 0, None, b["wq"], wT)
            if taps == 9:
                Q.qsync_conv3x3_wflip(b["wq"], N, C, b["wqbT"])

    want = buffers()
    separate(want, ws(need), ws(need))
    wx, ww = ws(need), ws(need)
    for second in (ww, wx):
        b = buffers()
        Q.qsync_convert_operands(code, x, M, C, b["amax"], w, N, taps, 8, g, b["sx"], b["ix"], b["ax"], b["xq"], b["xqT"], b["sw"],
                                 b["iw"], b["aw"], b["wq"], b["swb"], b["iwb"], b["wqbT"], wx, second)
        for name, t in want.items():
            if t is not None:
                assert_bits_equal(host(b[name]), host(t), name)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("vectors", [2040, 2048, 2056, 4096, 4104, 6144, 6152, 8192])
@pytest.mark.parametrize("last", [False, True])
def test_maximum_of_a_whole_tensor_in_every_workgroup(dtype, vectors, last):
    """Around the multiples of 2048 16-byte vectors at which a workgroup that finds the maximum by itself requests more, by 512 threads (the
    tensor alone) and by 256 (beside weights with a scale per row): the maximum in the first or in the last element, codes and scale the
    oracle's bit for bit."""
    e = 16 // np.dtype(dtype).itemsize
    rows = e if vectors % 16 else 64
    cols = vectors * e // rows
    assert cols % 8 == 0 and rows * cols == vectors * e      # what the vector tiles take
    rng = np.random.default_rng(vectors)
    x = _data(rng, (rows, cols), dtype, sigma=0.3)
    x[(-1, -1) if last else (0, 0)] = dtype(-7.5)
    say("whole tensor", dtype.__name__, rows, cols, "last", last)
    so, io = orc.scales_from_amax(orc.absmax(x, "tensor"))
    want = orc.quantize_int(x, io, "tensor", "nearest")
    f = lambda n: torch.zeros(n, dtype=torch.float32, device="cuda")
    codes = lambda r, c: torch.full((r, c), 99, dtype=torch.int8, device="cuda")
    s, iv, am, q, qT = f(1), f(1), f(1), codes(rows, cols), codes(cols, rows)
    Q.qsync_absmax_quantize(dev(x), rows, cols, 8, Q.ROUND_NEAREST, 0, 0, s, iv, am, q, qT, ws(Q.qsync_absmax_quantize_workspace_bytes(rows, cols)))
    N = 48
    w = _data(rng, (N, cols), np.float32, sigma=0.02)
    s2, q2, q2T, wq, wqT = f(1), codes(rows, cols), codes(cols, rows), codes(N, cols), codes(cols, N)
    need = max(Q.qsync_absmax_workspace_bytes(rows, cols, Q.PER_TENSOR), Q.qsync_absmax_workspace_bytes(N, cols, Q.PER_COL))
    sw = f(N)
    Q.qsync_convert_operands(Q.INT8, dev(x), rows, cols, None, dev(w), N, 1, 8, Q.PER_ROW, s2, f(1), f(1), q2, q2T, sw, f(N), f(N), wq, f(cols),
                             f(cols), wqT, ws(need), ws(need))
    for what, gs, gq, gqT in (("alone", s, q, qT), ("beside weights", s2, q2, q2T)):
        assert_bits_equal(host(gs), so, "scale " + what)
        assert_bits_equal(host(gq), want, "codes " + what)
        assert_bits_equal(host(gqT), want.T, "transposed codes " + what)
    wo, wi = orc.scales_from_amax(orc.absmax(w, "row"))
    assert_bits_equal(host(sw), wo, "weight scales")
    assert_bits_equal(host(wq), orc.quantize_int(w, wi, "row", "nearest"), "weight codes")


def test_absmax_quantize_all_zero_and_lower_bits():
    w = ws(Q.qsync_absmax_quantize_workspace_bytes(128, 256))
    z = torch.zeros(64, 128, dtype=torch.float16, device="cuda")
    s, iv, am = empty(1, torch.float32), empty(1, torch.float32), empty(1, torch.float32)
    q = torch.full((64, 128), 99, dtype=torch.int8, device="cuda")
    Q.qsync_absmax_quantize(z, 64, 128, 8, Q.ROUND_NEAREST, 0, 0, s, iv, am, q, None, w)
    torch.cuda.synchronize()
    assert s.item() == 1.0 and iv.item() == 1.0 and am.item() == 0.0 and int(q.abs().max().item()) == 0
    rng = np.random.default_rng(8)
    x = _data(rng, (128, 256), np.float32)
    so, io = orc.scales_from_amax(orc.absmax(x, "tensor"), 5)
    want = orc.quantize_int(x, io, "tensor", "stochastic", 9, 9, bits=5)
    q = torch.empty(128, 256, dtype=torch.int8, device="cuda")
    qT = torch.empty(256, 128, dtype=torch.int8, device="cuda")
    Q.qsync_absmax_quantize(dev(x), 128, 256, 5, Q.ROUND_STOCHASTIC, 9, 9, s, iv, am, q, qT, w)
    torch.cuda.synchronize()
    assert_bits_equal(host(s), so, "scale, 5 bits")
    assert_bits_equal(host(q), want, "codes, 5 bits")
    assert_bits_equal(host(qT), want.T, "transposed codes, 5 bits")


@pytest.mark.parametrize("src", [torch.float16, torch.float32])
@pytest.mark.parametrize("rows,cols,ld", [(8, 8, 8), (72, 64, 64), (248, 72, 88), (264, 136, 136), (4099, 8, 8), (8192, 1024, 1024),
                                          (8200, 256, 264), (8201, 256, 256), (8191, 264, 264), (31, 67656, 67656), (16401, 256, 256)])
def test_binary16_copies_by_every_route(src, rows, cols, ld):
    """Row-major and transposed binary16 copies, alone and together: patches, tiles and single elements on both sides of
    their limits (2^21 and 2^23 elements, whole and partial patches, row counts off 8), strided sources."""
    say("binary16 copies", src, rows, cols, ld)
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    x = torch.randn(rows, ld, device="cuda", generator=g).to(src)
    want = x[:, :cols].half()
    for want_q, want_t in ((True, False), (False, True), (True, True)):
        q = torch.full((rows, cols), 9.0, dtype=torch.float16, device="cuda") if want_q else None
        qT = torch.full((cols, rows), 9.0, dtype=torch.float16, device="cuda") if want_t else None
        Q.qsync_quantize(x, rows, cols, ld, Q.FP16, 0, 0, 0, 0, 0, None, q, qT)
        assert q is None or torch.equal(q, want)
        assert qT is None or torch.equal(qT, want.t())


@pytest.mark.parametrize("rnd", ["nearest", "stochastic"])
@pytest.mark.parametrize("rows,cols", [(1, 8), (1, 16384), (3, 65536), (15, 26216), (24, 336), (24, 344), (24, 680), (24, 688),
                                       (40, 4912), (40, 4920), (17, 23128), (17, 23136), (129, 248), (129, 256), (127, 264),
                                       (24, 2728), (24, 2736)])
def test_transposed_codes_of_odd_row_counts_by_every_route(rows, cols, rnd):
    """Row counts that are no multiple of 16, on both sides of each limit between one element per thread and tiles, and
    between one call's fused forms and the two separate passes: bits of the oracle either way."""
    rng = np.random.default_rng(rows + cols)
    x = _data(rng, (rows, cols), np.float16, sigma=0.3)
    so, io = orc.scales_from_amax(orc.absmax(x, "tensor"))
    want = orc.quantize_int(x, io, "tensor", rnd, 3, 17)
    say("odd rows", rows, cols, rnd)
    w = ws(Q.qsync_absmax_quantize_workspace_bytes(rows, cols))
    s, iv = empty(1, torch.float32), empty(1, torch.float32)
    for fused in (True, False):
        q = torch.full((rows, cols), 99, dtype=torch.int8, device="cuda")
        qT = torch.full((cols, rows), 99, dtype=torch.int8, device="cuda")
        if fused:
            Q.qsync_absmax_quantize(dev(x), rows, cols, 8, RND[rnd], 3, 17, s, iv, None, q, qT, w)
            assert_bits_equal(host(s), so, "scale")
            assert_bits_equal(host(iv), io, "inverse scale")
            assert int(w[:4].view(torch.int32).item()) == 0       # the arrival counter is left at zero
        else:
            Q.qsync_quantize(dev(x), rows, cols, cols, Q.INT8, 8, Q.PER_TENSOR, RND[rnd], 3, 17, iv, q, qT)
        assert_bits_equal(host(q), want, "codes")
        assert_bits_equal(host(qT), want.T, "transposed codes")


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("rows,cols", [(1, 8), (63, 120), (65, 136), (45, 1024), (128, 256), (129, 256), (130, 520),
                                       (8208, 1024)])
def test_transposed_codes_at_the_edges_of_the_tiles(dtype, rows, cols):
    """Codes and transposed codes of the tiled quantizer around its 64 and 128-row tiles, with row counts that leave the
    transposed copy unaligned, on both sides of the one-launch size, and of a strided input: bits of the oracle."""
    rng = np.random.default_rng(rows * 10007 + cols)
    x = _data(rng, (rows, cols), dtype, sigma=0.3)
    so, io = orc.scales_from_amax(orc.absmax(x, "tensor"))
    want = orc.quantize_int(x, io, "tensor", "stochastic", 5, 99)
    say("tile edges", dtype.__name__, rows, cols)
    s, iv, am = empty(1, torch.float32), empty(1, torch.float32), empty(1, torch.float32)
    q = torch.full((rows, cols), 99, dtype=torch.int8, device="cuda")
    qT = torch.full((cols, rows), 99, dtype=torch.int8, device="cuda")
    Q.qsync_absmax_quantize(dev(x), rows, cols, 8, Q.ROUND_STOCHASTIC, 5, 99, s, iv, am, q, qT,
                            ws(Q.qsync_absmax_quantize_workspace_bytes(rows, cols)))
    assert_bits_equal(host(s), so, "scale")
    assert_bits_equal(host(iv), io, "inverse scale")
    assert_bits_equal(host(q), want, "codes")
    assert_bits_equal(host(qT), want.T, "transposed codes")
    wide = torch.zeros(rows, cols + 16, dtype=dev(x).dtype, device="cuda")      # rows 16 elements apart
    wide[:, :cols] = dev(x)
    q.fill_(99), qT.fill_(99)
    Q.qsync_quantize(wide, rows, cols, cols + 16, Q.INT8, 8, Q.PER_TENSOR, Q.ROUND_STOCHASTIC, 5, 99, iv, q, qT)
    assert_bits_equal(host(q), want, "codes of the strided input")
    assert_bits_equal(host(qT), want.T, "transposed codes of the strided input")


@pytest.mark.parametrize("offset", [0, 4, 1])
@pytest.mark.parametrize("rows,cols", [(132, 136), (300, 256), (190, 128)])
def test_transposed_codes_of_rows_off_sixteen(rows, cols, offset):
    """Transposed copies whose columns are no multiple of 16 bytes leave as dwords (rows a multiple of four, aligned copy) or
    bytes (neither): bits of the oracle, and nothing written around them."""
    rng = np.random.default_rng(rows + cols + offset)
    x = _data(rng, (rows, cols), np.float16, sigma=0.3)
    so, io = orc.scales_from_amax(orc.absmax(x, "tensor"))
    want = orc.quantize_int(x, io, "tensor", "nearest")
    say("rows off sixteen", rows, cols, offset)
    room = torch.full((rows * cols + 64,), 99, dtype=torch.int8, device="cuda")
    qT = room[16 + offset:16 + offset + rows * cols].view(cols, rows)
    q = torch.full((rows, cols), 99, dtype=torch.int8, device="cuda")
    Q.qsync_quantize(dev(x), rows, cols, cols, Q.INT8, 8, Q.PER_TENSOR, Q.ROUND_NEAREST, 0, 0, dev(io), q, qT)
    assert_bits_equal(host(q), want, "codes")
    assert_bits_equal(host(qT), want.T, "transposed codes")
    around = host(room)
    assert (around[:16 + offset] == 99).all() and (around[16 + offset + rows * cols:] == 99).all()


@pytest.mark.parametrize("N,K", [(16, 8), (48, 136), (1040, 72), (2064, 16), (64, 2184)])
def test_weight_scales_over_every_batch_of_partial_maxima(N, K):
    """Both sets of scales and codes of the two-launch weight conversion where the folds run over one partial maximum, part of a
    batch, and several batches (over 16 row tiles, over 16 tile columns): bits of the oracle."""
    rng = np.random.default_rng(N * 31 + K)
    w = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    say("partial maxima", N, K)
    f = lambda n: torch.zeros(n, dtype=torch.float32, device="cuda")
    sw, iw, aw, swb, iwb = f(N), f(N), f(N), f(K), f(K)
    wq = torch.empty((N, K), dtype=torch.int8, device="cuda")
    wqbT = torch.empty((K, N), dtype=torch.int8, device="cuda")
    Q.qsync_prepare_weights(dev(w), N, K, 8, sw, iw, aw, wq, swb, iwb, wqbT, ws(Q.qsync_absmax_workspace_bytes(N, K, Q.PER_COL)))
    for gran, s, iv, got in (("row", sw, iw, host(wq)), ("col", swb, iwb, host(wqbT).T)):
        so, io = orc.scales_from_amax(orc.absmax(w, gran))
        assert_bits_equal(host(s), so, gran + " scales")
        assert_bits_equal(host(iv), io, gran + " inverse scales")
        assert_bits_equal(got, orc.quantize_int(w, io, gran, "nearest"), gran + " codes")


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("rows", [3, 4097])
def test_row_maxima_around_the_loads_of_a_lane(dtype, rows):
    """Rows of one, two and more vectors a lane (64 lanes a row, 256 below 4096 rows), whole and with a remainder, the maximum in
    the first, the last vector's or the very last element: scales of the oracle bit for bit."""
    lanes, e = (64 if rows >= 4096 else 256), 16 // np.dtype(dtype).itemsize
    for nvec in (1, lanes - 1, lanes, lanes + 1, 2 * lanes, 2 * lanes + 1, 4 * lanes, 4 * lanes + 1):
        cols = nvec * e
        x = _data(np.random.default_rng(rows + nvec), (rows, cols), dtype, sigma=0.1)
        x[0, 0], x[rows // 2, cols - e], x[rows - 1, cols - 1] = dtype(-5), dtype(6), dtype(-7)
        say("row maxima", dtype.__name__, rows, cols)
        so, io = orc.scales_from_amax(orc.absmax(x, "row"))
        s, iv, am = (empty(rows, torch.float32) for _ in range(3))
        Q.qsync_absmax_scale(dev(x), rows, cols, cols, Q.PER_ROW, 8, s, iv, am, None, ws(Q.qsync_absmax_workspace_bytes(rows, cols, Q.PER_ROW)))
        assert_bits_equal(host(s), so, "scale")
        assert_bits_equal(host(iv), io, "inverse scale")
