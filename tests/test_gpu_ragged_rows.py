"""GPU parity of the elementwise operators on short, ragged, channel-last and unaligned rows: every shape
class of the periodic and flat kernels (few and many vectors per period, one and several spans, one channel per
element, tails of one to three elements), against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403

SHAPES = [
    (5000, 3, 1), (700, 45, 1), (4097, 64, 1), (300, 1028, 1), (37, 5001, 1),   # channel-last, period below and above a workgroup
    (90, 5, 3), (64, 9, 2), (40, 7, 59), (33, 300, 7), (16, 6, 196),            # short rows, odd periods (taken two or four times)
    (1, 89, 5354), (2, 50, 761), (3, 1111, 3), (1, 4099, 1), (2, 3, 2),         # the pattern does not come back: flat
    (9, 2, 1023), (5, 24, 1001), (1, 1, 4101), (70, 1, 3), (2, 1500, 33), (3, 17000, 5), (17, 9000, 1),
]


def _view(x, offset):
    """The same values in a GPU tensor that starts `offset` elements into its allocation."""
    base = torch.empty(x.size + offset, dtype=getattr(torch, x.dtype.name), device=DEV)
    v = base[offset:].view(x.shape)
    v.copy_(torch.from_numpy(x))
    return v


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("offset", [0, 1])
def test_every_operator_on_ragged_rows(shape, offset):
    rng = np.random.default_rng(abs(hash((shape, offset))) % 2 ** 31)
    C = shape[1]
    x = (rng.standard_normal(shape) * 2).astype(np.float32)
    special = np.array([np.nan, np.inf, -np.inf, -0.0, 0.125, 3e38, 1e-40], np.float32)
    x.reshape(-1)[rng.permutation(x.size)[: 7]] = special[: x.size]
    scale = rng.uniform(0.01, 0.05, C).astype(np.float32)
    zp = rng.integers(-20, 20, C).astype(np.int32)
    dx, ds, dz, q = _view(x, offset), dev(scale), dev(zp), hago.QType(hago.I8)
    out = lambda dt: _view(np.full(shape, 77, dt), offset)  # noqa: E731
    want = ref.simquant(x, scale, zp, -128, 127)
    codes = ref.quantize(x, scale, zp, -128, 127)
    assert_same_bits(host(hago.simquant(dx, ds, dz, q, out=out(np.float32))), want, f"simquant {shape}")
    assert_same_bits(host(hago.simquant_wrap(dx, ds, dz, q)), ref.simquant_wrap(x, scale, zp, 8, True, -128, 127), f"wrap {shape}")
    assert_same(host(hago.quantize(dx, ds, dz, q, out=out(np.int8))).astype(np.int32), codes, f"quantize {shape}")
    y, c = hago.simquant_codes(dx, ds, dz, q, out=out(np.float32), out_codes=out(np.int8))
    assert_same_bits(host(y), want, f"simquant_codes {shape}")
    assert_same(host(c).astype(np.int32), codes, f"codes {shape}")
    for dt, qt in ((np.int8, q), (np.int16, hago.QType(hago.I16)), (np.int32, hago.QType(hago.I32, 20, True))):
        got = hago.dequantize(_view(codes.astype(dt), offset), qt, ds, dz)
        assert_same_bits(host(got), ref.dequantize(codes, scale, zp), f"dequantize {shape} {dt.__name__}")
    sc2 = np.stack([scale, scale * np.float32(1.7), scale[::-1]]).astype(np.float32)
    zp2 = np.stack([zp, zp + 1, -zp]).astype(np.int32)
    lo, hi = [-128, -8, -64], [127, 7, 63]
    got = host(hago.simquant_batched(dx, dev(sc2), dev(zp2), q, lo, hi))
    for b in range(3):
        assert_same_bits(got[b], ref.simquant(x, sc2[b], zp2[b], lo[b], hi[b]), f"candidate {b} {shape}")
    for pc in (True, False):
        assert_same_bits(host(hago.absmax(dx, pc)), ref.absmax(x, pc), f"absmax {shape} {pc}")
    acc = rng.integers(-2 ** 20, 2 ** 20, shape).astype(np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, C).astype(np.int32)
    shift = rng.integers(8, 14, C).astype(np.int32)
    for rounding in (0, 1):
        got = hago.requantize(_view(acc, offset), gpu_requant(mult, shift, rounding=rounding), out=out(np.int8))
        assert_same(host(got), ref.requantize(acc, ref_requant(mult, shift, rounding=rounding)), f"requantize {shape}")
    a16 = (acc >> 6).astype(np.int16)
    assert_same(host(hago.requantize(_view(a16, offset), gpu_requant(mult, shift))), ref.requantize(a16, ref_requant(mult, shift)),
                f"requantize int16 {shape}")


def test_requantize_int16_many_wavefronts():
    """A chip full of wavefronts, a few times: each lane's shift is its own wherever its registers lie."""
    n = 2 ** 25 + 5
    a = np.random.default_rng(5).integers(-30000, 30000, (1, 1, n)).astype(np.int16)
    want = ref.requantize(a, ref_requant([2 ** 30], [7]))
    da, rq = dev(a), gpu_requant([2 ** 30], [7])
    for _ in range(4):
        assert_same(host(hago.requantize(da, rq)), want, "int16, flat")


@pytest.mark.parametrize("shape", [(70, 200, 1), (5000, 129, 1), (33, 131, 3), (300, 768, 1), (16, 100, 49), (1100, 4001, 1), (20000, 33, 1),
                                   (64, 43, 3)])
def test_absmax_by_slabs_of_channels(shape):
    """Patterns of more than 32 vectors, whole and ragged slabs of 16 vectors, channels that run on over several elements."""
    rng = np.random.default_rng(sum(shape))
    x = rng.normal(0, 1, shape).astype(np.float32)
    x[:, ::5] *= -7.0
    x[0, 0, 0] = np.nan
    x[-1, -1, -1] = -np.inf
    x[:, shape[1] // 2] = 0.0
    assert_same_bits(host(hago.absmax(dev(x))), ref.absmax(x, True), f"absmax {shape}")
