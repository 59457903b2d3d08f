"""What a convolution call may bring to any kernel that serves it: tensors that start on any byte, power-of-two scales (no
multiplier), 24-bit accumulators, one scale for all channels.  Every wavefront shape of the two kernels that take any
geometry, the kernels of 1x1 and 3x3 layers, and the one that streams channel-last tensors (whose operands are aligned), against
the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403

CASES = [
    # B C H W O KH KW stride pad
    (2, 3, 31, 37, 20, 7, 7, (2, 2), (3, 3)),      # few channels
    (2, 17, 7, 9, 33, 3, 3, (1, 1), (1, 1)),
    (2, 24, 14, 15, 70, 1, 1, (2, 2), (0, 0)),
    (1, 64, 13, 12, 65, 5, 5, (1, 1), (2, 2)),
    (3, 48, 9, 8, 40, 1, 1, (1, 1), (0, 0)),       # the 1x1 kernels' own
    (2, 32, 9, 12, 72, 3, 3, (1, 1), (1, 1)),      # the 3x3 kernel's own
    (2, 146, 12, 13, 24, 3, 3, (1, 1), (1, 1)),    # several chunks of channels
]
# kernel (hook), wavefront shape
KERNELS = [(0, -1)] + [(3, s) for s in (-1, 0, 1, 2)] + [(4, s) for s in (0, 1, 2, 3)] + [(5, s) for s in (0, 1)]


def _at(x, offset, fill=None):
    """A device tensor of x's values (or of `fill`) that starts `offset` bytes into its allocation; and the allocation."""
    raw = torch.full((x.nbytes + offset + 16,), 0x5A, dtype=torch.uint8, device=DEV)
    t = raw[offset:offset + x.nbytes].view(getattr(torch, x.dtype.name)).view(x.shape)
    if fill is None:
        t.copy_(torch.from_numpy(x))
    return t, raw


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_forms_of_a_call(case, kernel, layout, gemm_path):
    B, C, H, W, O, KH, KW, stride, pad = case
    path, shape = kernel
    if path == 4 and shape == 3 and layout == "nhwc" and C >= 16:  # (three shapes)
        return
    if path == 5 and (layout == "nchw" or C % 16 != 0):
        return
    rng = np.random.default_rng(C * 100 + O + KH)
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    to = (lambda x: x) if layout == "nchw" else (lambda x: np.ascontiguousarray(x.transpose(0, 2, 3, 1)))
    w = to(rng.integers(-127, 128, (O, C, KH, KW)).astype(np.int8))
    bias = rng.integers(-2 ** 24, 2 ** 24, O).astype(np.int32)     # (24-bit sums wrap)
    mult = rng.integers(2 ** 30, 2 ** 31, O).astype(np.int32)
    shift = rng.integers(11, 15, O).astype(np.int32)
    i8_g, u8_g = hago.QType(hago.I8), hago.QType(hago.U8, 8, False, 7)
    forms = [   # accumulator, multiplier, shift, tie rule, unsigned output; none: raw
        (hago.I32, ref.I32, None, shift, 0, True), (hago.I32, ref.I32, None, np.where(shift > 12, 0, shift), 1, False),
        (hago.I24, ref.I24, mult, shift, 0, False), (hago.I24, ref.I24, None, shift, 0, True),
        (hago.I32, ref.I32, mult[:1], shift[:1], 0, True), (hago.I24, ref.I24, "raw", None, 0, False),
        (hago.I16, ref.I16, mult, shift - 8, 0, False), (hago.I16, ref.I16, "raw", None, 0, False)]
    gemm_path(path)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, shape)
    try:
        for n, (acc_g, acc_r, m, s, rounding, out_u8) in enumerate(forms):
            a = to(rng.integers(0, 256, (B, C, H, W)).astype(np.uint8) if n % 2 else rng.integers(-128, 128, (B, C, H, W)).astype(np.int8))
            za = (0, 131, -5, 0)[n % 4]
            raw = isinstance(m, str)
            rq_r = None if raw else ref.Requant(m, s, out_dtype=ref.U8 if out_u8 else ref.I8, out_zero_point=7 if out_u8 else 0,
                                                clip_lo=0 if out_u8 else -128, clip_hi=255 if out_u8 else 127, rounding=rounding)
            rq_g = None if raw else hago.Requant(None if m is None else dev(m), dev(s.astype(np.int32)), u8_g if out_u8 else i8_g, rounding=rounding)
            want = ref.qconv2d(a, za, w, bias, lay_r, stride, pad, 1, acc_r, rq_r)
            (da, _), (dw, _) = (_at(a, 0), _at(w, 0)) if path == 5 else (_at(a, 1 + n % 3), _at(w, 3 - n % 3))
            step = want.dtype.itemsize
            out, around = _at(want, step * (1 + n % 3), fill=True)
            got = hago.qconv2d(da, act_qtype(a, za), dw, i8_g, dev(bias), lay_g, stride, pad, 1, acc_g, rq_g, out=out)
            assert_same(host(got), want, f"form {n}, {kernel}")
            edge = step * (1 + n % 3)
            around = host(around)
            assert (around[:edge] == 0x5A).all() and (around[edge + want.nbytes:] == 0x5A).all(), "wrote beside the output"
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)
