"""Stores that go through the L2: elementwise spans of whole lines and of broken ones on both sides of their size rule, many
candidates on both sides of theirs, dense tiles of every width at rows that begin with a line or anywhere, NCHW layers on both
sides of their lines."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403


# (odd, even and multiple-of-four periods; spans cut to whole lines or not; below and above 2.5 million elements)
@pytest.mark.parametrize("shape", [(900, 45, 1), (60001, 45, 1), (38500, 65, 1), (39000, 65, 1), (5000, 33, 1), (3000, 39, 1), (2500, 22, 3)])
def test_spans(shape):
    rng = np.random.default_rng(shape[0])
    C = shape[1]
    x = (rng.standard_normal(shape) * 2).astype(np.float32)
    scale, zp = rng.uniform(0.01, 0.05, C).astype(np.float32), rng.integers(-20, 20, C).astype(np.int32)
    dx, ds, dz, q = dev(x), dev(scale), dev(zp), hago.QType(hago.I8)
    want, codes = ref.simquant(x, scale, zp, -128, 127), ref.quantize(x, scale, zp, -128, 127)
    assert_same_bits(host(hago.simquant(dx, ds, dz, q)), want, "simquant")
    y, c = hago.simquant_codes(dx, ds, dz, q)
    assert_same_bits(host(y), want, "simquant_codes")
    assert_same(host(c).astype(np.int32), codes, "codes")
    assert_same(host(hago.quantize(dx, ds, dz, q)).astype(np.int32), codes, "quantize")
    assert_same_bits(host(hago.dequantize(c, q, ds, dz)), ref.dequantize(codes, scale, zp), "dequantize")


def test_spans_of_65_channels_below_the_rule():
    assert 38400 * 65 < 2500000 < 38500 * 65
    test_spans((38400, 65, 1))


@pytest.mark.parametrize("outer", [31, 32])   # 8 candidates of 2^21 + 2^16 (outer - 32) elements x 4: 2^26 results and just below
def test_candidates(outer):
    g = torch.Generator(device=DEV)
    g.manual_seed(outer)
    x = torch.randn((outer, 64, 4096), generator=g, device=DEV)
    scales = torch.rand((8, 64), generator=g, device=DEV) * 0.04 + 0.01
    zps = torch.randint(-9, 10, (8, 64), generator=g, device=DEV, dtype=torch.int32)
    lo, hi = [-128, -64, -32, -16, -8, -8, -4, -2], [127, 63, 31, 15, 7, 7, 3, 1]
    for n in (8, 1) if outer == 31 else (8,):
        got = hago.simquant_batched(x, scales[:n].contiguous(), zps[:n].contiguous(), hago.QType(hago.I8), lo[:n], hi[:n])
        for b in range(n):
            one = hago.simquant(x, scales[b].contiguous(), zps[b].contiguous(), hago.QType(hago.I8), lo[b], hi[b])
            assert torch.equal(got[b].view(torch.int32), one.view(torch.int32)), (n, b)
    part = host(x[:1, :2]).copy()
    assert_same_bits(host(got[0][:1, :2]), ref.simquant(part, host(scales[0][:2]), host(zps[0][:2]), lo[0], hi[0]), "oracle")


@pytest.mark.parametrize("outer", [32, 33])   # 8 candidates of 2^18 elements each: 2^26 results, which go through the L2, and more, which do not
def test_candidates_of_both_forms(outer):
    g = torch.Generator(device=DEV)
    g.manual_seed(outer)
    x = torch.randn((outer, 64, 4096), generator=g, device=DEV)
    scales = torch.rand((8, 64), generator=g, device=DEV) * 0.04 + 0.01
    zps = torch.randint(-9, 10, (8, 64), generator=g, device=DEV, dtype=torch.int32)
    lo, hi = [-128, -64, -32, -16, -8, -8, -4, -2], [127, 63, 31, 15, 7, 7, 3, 1]
    assert (x.numel() * 8 <= 1 << 26) == (outer == 32)
    for n in (8, 1):
        got = hago.simquant_batched(x, scales[:n].contiguous(), zps[:n].contiguous(), hago.QType(hago.I8), lo[:n], hi[:n])
        for b in range(n):
            one = hago.simquant(x, scales[b].contiguous(), zps[b].contiguous(), hago.QType(hago.I8), lo[b], hi[b])
            assert torch.equal(got[b].view(torch.int32), one.view(torch.int32)), (n, b)
            for o, c in ((0, 0), (outer - 1, 62)):   # the first rows and the last
                part = host(x[o:o + 1, c:c + 2]).copy()
                want = ref.simquant(part, host(scales[b][c:c + 2]), host(zps[b][c:c + 2]), lo[b], hi[b])
                assert_same_bits(host(got[b][o:o + 1, c:c + 2]), want, f"oracle {n, b, o, c}")


@pytest.mark.parametrize("n", [64, 72, 128, 129, 192, 200, 1001])
@pytest.mark.parametrize("m, k, off", [(700, 128, 0), (700, 128, 16), (700, 128, 1), (2100, 768, 0)])
def test_dense_rows(n, m, k, off):
    rng = np.random.default_rng(n * 1000 + m + off)
    a, w = rng.integers(0, 256, (m, k)).astype(np.uint8), rng.integers(-127, 128, (n, k)).astype(np.int8)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, n).astype(np.int32), rng.integers(6, 10, n).astype(np.int32)
    guard = torch.full((m * n + off + 64,), 77, dtype=torch.int8, device=DEV)
    out = guard[off:off + m * n].view(m, n)
    hago.qdense(dev(a), act_qtype(a, 128), dev(w), hago.QType(hago.I8), None, hago.I32, gpu_requant(mult, shift), out=out)
    assert_same(host(out), ref.qdense(a, 128, w, None, ref.I32, ref_requant(mult, shift)), f"{m}x{k}->{n}")
    assert int((host(guard[:off]) != 77).sum()) == 0 and int((host(guard[off + m * n:]) != 77).sum()) == 0


# NCHW layers: images that begin with a line, at 16 bytes, at 4 and anywhere; few and many workgroups; a tile's end inside sixteen pixels
@pytest.mark.parametrize("case", [(2, 32, 33, 36, 40, 3), (3, 64, 15, 16, 72, 3), (64, 64, 19, 20, 40, 3), (24, 32, 56, 56, 33, 3),
                                  (24, 32, 28, 28, 70, 3), (9, 32, 13, 13, 70, 1), (7, 24, 20, 20, 33, 1), (5, 68, 31, 30, 40, 1),
                                  (4, 32, 41, 41, 36, 1), (8, 32, 56, 56, 100, 1)])
def test_nchw_layers(case):
    B, C, H, W, O, k = case
    rng = np.random.default_rng(1000 * W + O)
    w = rng.integers(-127, 128, (O, C, k, k)).astype(np.int8)
    a = rng.integers(0, 256, (B, C, H, W)).astype(np.uint8)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, O).astype(np.int32), rng.integers(7, 12, O).astype(np.int32)
    geo, rgeo = (hago.NCHW, (1, 1), (k // 2, k // 2), 1), (ref.NCHW, (1, 1), (k // 2, k // 2), 1)
    raw = ref.qconv2d(a, 131, w, None, *rgeo)
    forms = [(hago.I32, None, torch.int32, raw), (hago.I16, None, torch.int16, raw.astype(np.int16))]
    for clip, acc, racc in (((-128, 127), hago.I32, ref.I32), ((-100, 90), hago.I32, ref.I32), ((-128, 127), hago.I16, ref.I16)):
        want = ref.qconv2d(a, 131, w, None, *rgeo, racc, ref_requant(mult, shift, False, -3, clip))
        forms.append((acc, gpu_requant(mult, shift, False, -3, clip), torch.int8, want))
    args = (dev(a), act_qtype(a, 131), dev(w), hago.QType(hago.I8), None, *geo)
    for acc, rq, dtype, want in forms:
        for off in (0, 1, 16):
            got = into_guard(lambda out: hago.qconv2d(*args, acc, rq, out=out), raw.shape, dtype, off)
            assert_same(got, want, f"{case} {dtype} off {off}")


# depthwise layers on both sides of 11 MB of results: by the dword, by four rows (every remainder of a quarter's rows, images that end
# inside sixteen bytes), rows off dwords left in the L2 or not, segments
@pytest.mark.parametrize("case", [(2, 70, 45, 44), (57, 100, 45, 44), (60, 60, 57, 60), (65, 57, 49, 64), (40, 96, 64, 48), (130, 150, 16, 36),
                                  (110, 200, 13, 52), (62, 80, 43, 53), (75, 60, 50, 51), (9, 11, 50, 41), (120, 60, 40, 41), (3, 9, 40, 113)])
def test_depthwise_rows(case):
    B, C, H, W = case
    rng = np.random.default_rng(1000 * W + H)
    w = rng.integers(-127, 128, (C, 1, 3, 3)).astype(np.int8)
    a = rng.integers(-127, 128, (B, C, H, W)).astype(np.int8)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, C).astype(np.int32), rng.integers(7, 12, C).astype(np.int32)
    want = ref.qconv2d(a, 0, w, None, ref.NCHW, (1, 1), (1, 1), C, ref.I32, ref_requant(mult, shift))
    args = (dev(a), act_qtype(a, 0), dev(w), hago.QType(hago.I8), None, hago.NCHW, (1, 1), (1, 1), C, hago.I32, gpu_requant(mult, shift))
    for off in (0, 4, 1):
        assert_same(into_guard(lambda out: hago.qconv2d(*args, out=out), a.shape, torch.int8, off), want, f"{case} off {off}")


# layers of more than 11 MB of results, of whose rows four meet in LDS, in every kind of codes and form of the arithmetic
@pytest.mark.parametrize("case", [(57, 100, 45, 44), (40, 96, 64, 48)])
@pytest.mark.parametrize("act_u8", [False, True])
def test_depthwise_four_rows(case, act_u8):
    B, C, H, W = case
    assert B * C * H * W > 11e6
    rng = np.random.default_rng(1000 * W + H + act_u8)
    w = rng.integers(-127, 128, (C, 1, 3, 3)).astype(np.int8)
    a = rng.integers(0, 256, (B, C, H, W)).astype(np.uint8) if act_u8 else rng.integers(-127, 128, (B, C, H, W)).astype(np.int8)
    za = 131 if act_u8 else 0
    geo, rgeo = (hago.NCHW, (1, 1), (1, 1), C), (ref.NCHW, (1, 1), (1, 1), C)
    sums = ref.qconv2d(a, za, w, None, *rgeo, ref.I32).reshape(B, C, H * W)
    da, dw = dev(a), dev(w)
    for acc, out_u8, z, clip, rounding, odd in (
            (hago.I32, False, -3, (-128, 127), 0, True), (hago.I32, True, 7, (0, 255), 0, False), (hago.I32, False, 0, (-100, 90), 0, True),
            (hago.I32, False, 5, (-128, 127), 1, False), (hago.I16, False, -3, (-128, 127), 0, True), (hago.I24, True, 7, (0, 255), 0, False)):
        mult, shift = rng.integers(2 ** 30, 2 ** 31, C).astype(np.int32), rng.integers(7, 12, C).astype(np.int32)
        bias = rng.integers(-3000, 3000, C).astype(np.int32)
        if odd:   # single channels off the forms of the others
            shift[3], shift[C - 1], bias[5], bias[C - 2] = 0, 23, 2 ** 30 + 9, -2 ** 30 - 9
        bits = {hago.I32: 32, hago.I24: 24, hago.I16: 16}[acc]
        wrapped = ((sums.astype(np.int64) + bias[:, None] + (1 << (bits - 1))) % (1 << bits) - (1 << (bits - 1))).astype(np.int32)
        want = ref.requantize(wrapped, ref_requant(mult, shift, out_u8, z, clip, rounding)).reshape(a.shape)
        got = into_guard(lambda out: hago.qconv2d(da, act_qtype(a, za), dw, hago.QType(hago.I8), dev(bias), *geo, acc,
                                                  gpu_requant(mult, shift, out_u8, z, clip, rounding=rounding), out=out),
                         a.shape, torch.uint8 if out_u8 else torch.int8, 4)
        assert_same(got, want, f"{case} u8={act_u8} {acc, out_u8, z, clip, rounding, odd}")
