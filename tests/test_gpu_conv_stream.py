"""GPU parity of the channel-last convolution that streams the caller's tensors into LDS, in every tile shape, against the
oracle: reductions that end inside a stage, stages that hold one tap and several, filters that hang over every edge and lie
outside the image altogether, images of which a tile holds several and images too large for a pixel's place in one to be a
multiplication, channel and pixel counts off the tile, zero points that do and do not equal the zeros that loads out of range
leave, before the flip and behind it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

CASES = [
    # B C H W O KH KW stride pad
    (1, 16, 4, 5, 3, 1, 1, (2, 2), (0, 0)),         # one chunk
    (2, 16, 7, 9, 33, 3, 3, (1, 1), (1, 1)),        # a stage of four taps
    (3, 48, 6, 5, 64, 3, 3, (1, 1), (1, 1)),        # taps that straddle stages
    (2, 64, 9, 9, 70, 3, 3, (2, 2), (1, 1)),        # a tap a stage
    (1, 128, 13, 11, 65, 3, 3, (1, 1), (1, 1)),
    (5, 80, 7, 7, 130, 5, 5, (1, 1), (2, 2)),
    (2, 32, 6, 8, 5, 3, 3, (1, 1), (4, 4)),         # filters outside the image altogether
    (1, 32, 5, 4, 12, 3, 2, (1, 2), (0, 1)),
    (1, 64, 40, 41, 64, 1, 3, (1, 1), (0, 1)),
    (40, 192, 1, 3, 20, 3, 3, (1, 1), (1, 1)),      # tiles of many images
    (70, 64, 1, 1, 20, 1, 1, (1, 1), (1, 1)),
    (1, 112, 17, 19, 64, 7, 7, (2, 2), (3, 3)),
    (1, 16, 1, 65540, 5, 1, 3, (1, 1), (0, 1)),     # 2^32 and more: pixels times pixels of an image, and of a row
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("shape", [0, 1])
def test_streamed_convolution(case, shape, gemm_path):
    B, C, H, W, O, KH, KW, stride, pad = case
    rng = np.random.default_rng(sum(case[:7]))
    w = rng.integers(-127, 128, (O, KH, KW, C)).astype(np.int8)
    bias = rng.integers(-10 ** 5, 10 ** 5, O).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(C * KH * KW)), 40.0)
    w_t, args, rargs = hago.QType(hago.I8), (hago.NHWC, stride, pad, 1), (ref.NHWC, stride, pad, 1)
    gemm_path(5)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, shape)
    try:
        for adt, za in ((np.uint8, 131), (np.uint8, 128), (np.uint8, 0), (np.int8, 0), (np.int8, -5)):
            a = (rng.integers(0, 256, (B, H, W, C)) if adt == np.uint8 else rng.integers(-128, 128, (B, H, W, C))).astype(adt)
            a_t, da, dw = act_qtype(a, za), dev(a), dev(w)
            if za == 0:
                assert_same(host(hago.qconv2d(da, a_t, dw, w_t, None, *args, hago.I16)), ref.qconv2d(a, za, w, None, *rargs, ref.I16), "raw 16")
                assert_same(host(hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args)), ref.qconv2d(a, za, w, bias, *rargs), f"raw {case}")
                continue
            for out_u8, z, clip, rounding in ((False, -3, (-128, 127), 0), (True, 10, (10, 255), 1)):
                want = ref.qconv2d(a, za, w, bias, *rargs, ref.I32, ref_requant(mult, shift, out_u8, z, clip, rounding))
                got = hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args, hago.I32, gpu_requant(mult, shift, out_u8, z, clip, rounding=rounding))
                assert_same(host(got), want, f"requantized {case} {adt} u8={out_u8}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)
