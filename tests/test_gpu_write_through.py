"""Stores that go through the L2: elementwise spans of whole lines and of broken ones on both sides of their size rule, many
candidates on both sides of theirs, and dense tiles of every width at rows that begin with a line or anywhere."""
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
