"""GPU parity of the NCHW 1x1 convolution of any size and alignment against the oracle: images of less than a tile and off
it, input channels off the 32 of a step, all in registers or in chunks, the reduction split over wavefronts, several
blocks of output channels per wavefront, every output mode."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

SIZES = [  # B C H W O
    (1, 4, 1, 4, 1), (3, 24, 1, 5, 33), (2, 32, 3, 3, 40), (1, 36, 7, 7, 32), (5, 64, 9, 9, 64), (2, 60, 11, 13, 70),
    (1, 68, 8, 16, 33), (2, 96, 10, 13, 96), (1, 100, 15, 15, 20), (2, 164, 12, 11, 65), (1, 576, 14, 14, 96),
    (3, 640, 5, 5, 31), (1, 324, 40, 41, 45), (9, 24, 57, 55, 144), (4, 80, 56, 57, 160), (1, 100, 46, 47, 1000),
    (2, 8, 1, 127, 6), (2, 40, 3, 43, 7), (1, 72, 4, 32, 5),
    # just more blocks than wavefronts of some or all variants run at once, and so two to four blocks each: small images, larger ones
    (1030, 68, 1, 4, 40), (1100, 68, 1, 5, 100), (1040, 36, 2, 3, 70), (1100, 64, 1, 4, 100), (1030, 68, 8, 16, 33),
]


@pytest.mark.parametrize("size", SIZES)
def test_pointwise_any_size(size):
    B, C, H, W, O = size
    rng = np.random.default_rng(C * 1000 + W)
    w = rng.integers(-127, 128, (O, C, 1, 1)).astype(np.int8)
    bias = rng.integers(-10 ** 4, 10 ** 4, O).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(C)), 40.0)
    args, rargs = (hago.NCHW, (1, 1), (0, 0), 1), (ref.NCHW, (1, 1), (0, 0), 1)
    w_t, dw = hago.QType(hago.I8), dev(w)
    for adt, za in ((np.uint8, 131), (np.int8, 0), (np.int8, -5)):
        a = (rng.integers(0, 256, (B, C, H, W)) if adt == np.uint8 else rng.integers(-128, 128, (B, C, H, W))).astype(adt)
        a_t, da = act_qtype(a, za), dev(a)
        if za == -5:  # a tensor that starts at an odd byte
            buf = torch.zeros(a.size + 1, dtype=torch.int8, device="cuda:0")
            buf[1:] = da.reshape(-1)
            da = buf[1:].reshape(da.shape)
        for acc, racc, out_u8, z, clip, rounding in ((hago.I32, ref.I32, False, -3, (-128, 127), 0), (hago.I32, ref.I32, True, 10, (10, 255), 1),
                                                     (hago.I16, ref.I16, False, 0, (-127, 127), 0)):
            want = ref.qconv2d(a, za, w, bias, *rargs, racc, ref_requant(mult, shift, out_u8, z, clip, rounding))
            got = hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args, acc, gpu_requant(mult, shift, out_u8, z, clip, rounding=rounding))
            assert_same(host(got), want, f"requantized {size} u8={out_u8} acc={acc}")
        assert_same(host(hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args)), ref.qconv2d(a, za, w, bias, *rargs), f"raw {size}")
        assert_same(host(hago.qconv2d(da, a_t, dw, w_t, None, *args, hago.I16)), ref.qconv2d(a, za, w, None, *rargs, ref.I16), f"raw 16 {size}")
