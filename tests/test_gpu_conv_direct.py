"""GPU parity of the one-launch convolution for any geometry, every wavefront shape, layout and output mode, against the
oracle: few and many channels, channel counts off every group size, tiles that span images, column segments, strides
beyond the kernel, quads of columns that hang over either edge, channels in several chunks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

CASES = [
    # B C H W O KH KW stride pad
    (2, 3, 31, 37, 20, 7, 7, (2, 2), (3, 3)),      # few channels, 4 bytes per pixel
    (1, 4, 9, 9, 70, 3, 3, (1, 1), (1, 1)),
    (3, 6, 11, 14, 33, 5, 5, (1, 1), (2, 2)),      # 8 bytes
    (2, 13, 8, 21, 65, 3, 3, (2, 2), (1, 1)),      # 16 bytes
    (5, 40, 7, 7, 45, 3, 3, (1, 1), (1, 1)),       # tiles span images
    (7, 65, 7, 9, 130, 1, 1, (1, 1), (0, 0)),
    (2, 24, 14, 15, 70, 1, 1, (2, 2), (0, 0)),     # stride beyond the kernel
    (1, 17, 13, 300, 9, 3, 3, (1, 1), (1, 1)),     # column segments
    (1, 33, 5, 530, 66, 3, 3, (2, 1), (1, 1)),
    (2, 146, 12, 13, 24, 3, 3, (1, 1), (1, 1)),    # several chunks
    (1, 300, 6, 5, 140, 5, 5, (1, 1), (2, 2)),
    (2, 64, 16, 16, 128, 3, 3, (2, 2), (1, 1)),
    (1, 20, 5, 4, 12, 3, 2, (1, 2), (0, 1)),
    (1, 32, 1, 64, 64, 1, 3, (1, 1), (0, 1)),      # one row
    (2, 18, 6, 8, 5, 3, 3, (1, 1), (4, 4)),        # padding wider than a quad
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("shape", [-1, 0, 1, 2])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_direct_convolution(case, shape, layout, gemm_path):
    B, C, H, W, O, KH, KW, stride, pad = case
    rng = np.random.default_rng(abs(hash(case)) % 2 ** 31)
    w = rng.integers(-127, 128, (O, C, KH, KW)).astype(np.int8)
    bias = rng.integers(-10 ** 5, 10 ** 5, O).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(C * KH * KW)), 40.0)
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    to = (lambda x: x) if layout == "nchw" else (lambda x: np.ascontiguousarray(x.transpose(0, 2, 3, 1)))
    w_t, wl = hago.QType(hago.I8), to(w)
    args, rargs = (lay_g, stride, pad, 1), (lay_r, stride, pad, 1)
    gemm_path(3)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, shape)
    try:
        for adt, za in ((np.uint8, 131), (np.int8, 0), (np.int8, -5)):
            a = to((rng.integers(0, 256, (B, C, H, W)) if adt == np.uint8 else rng.integers(-128, 128, (B, C, H, W))).astype(adt))
            a_t, da, dw = act_qtype(a, za), dev(a), dev(wl)
            assert_same(host(hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args)), ref.qconv2d(a, za, wl, bias, *rargs), f"raw {case}")
            if za == 0:
                assert_same(host(hago.qconv2d(da, a_t, dw, w_t, None, *args, hago.I16)), ref.qconv2d(a, za, wl, None, *rargs, ref.I16), "raw 16")
                continue
            for out_u8, z, clip, rounding in ((False, -3, (-128, 127), 0), (True, 10, (10, 255), 1)):
                want = ref.qconv2d(a, za, wl, bias, *rargs, ref.I32, ref_requant(mult, shift, out_u8, z, clip, rounding))
                got = hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args, hago.I32, gpu_requant(mult, shift, out_u8, z, clip, rounding=rounding))
                assert_same(host(got), want, f"requantized {case} u8={out_u8}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("layout,C,O,stride", [("nchw", 32, 37, 1), ("nchw", 128, 70, 1), ("nchw", 36, 70, 2), ("nchw", 38, 70, 2), ("nhwc", 48, 70, 2),
                                               ("nhwc", 40, 70, 2)])
def test_weights_at_any_byte(layout, C, O, stride, off, gemm_path):
    """3x3 weights loaded by descriptor (both one-launch kernels): tensors that start inside a dword, between other bytes,
    channel counts on both sides of the whole units, output channels off the block."""
    rng = np.random.default_rng(C + off)
    a, za = rng.integers(0, 256, (2, C, 12, 16)).astype(np.uint8), 131
    w, bias = rng.integers(-127, 128, (O, C, 3, 3)).astype(np.int8), rng.integers(-10 ** 5, 10 ** 5, O).astype(np.int32)
    if layout == "nhwc":
        a, w = (np.ascontiguousarray(x.transpose(0, 2, 3, 1)) for x in (a, w))
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    whole = torch.full((w.size + 32,), 77, dtype=torch.int8, device="cuda:0")
    dw = whole[16 + off: 16 + off + w.size].view(w.shape)
    dw.copy_(dev(w))
    want = ref.qconv2d(a, za, w, bias, lay_r, (stride, stride), (1, 1), 1)
    if stride == 2:
        gemm_path(3)
    got = hago.qconv2d(dev(a), act_qtype(a, za), dw, hago.QType(hago.I8), dev(bias), lay_g, (stride, stride), (1, 1), 1)
    assert_same(host(got), want, f"{layout} C={C} off {off}")
