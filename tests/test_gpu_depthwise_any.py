"""GPU parity of the depthwise 3 x 3 convolution of any size and alignment against the oracle: rows of every remainder,
rows of a few columns (channels share a tile), one tile and several along the row, tiles that span images, odd channel
counts, both layouts and strides, every output mode, and a window that reaches past the tensor's last row."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

SIZES = [  # B C H W
    (1, 1, 1, 4), (2, 3, 5, 5), (3, 5, 7, 7), (5, 4, 6, 8), (2, 7, 3, 9), (3, 6, 14, 14), (1, 3, 20, 15), (2, 2, 16, 16),
    (2, 3, 17, 17), (1, 5, 28, 28), (1, 2, 31, 31), (2, 3, 33, 32), (1, 3, 40, 33), (2, 5, 41, 41), (1, 2, 9, 61),
    (1, 3, 12, 62), (1, 2, 35, 63), (1, 2, 70, 65), (1, 3, 67, 69), (1, 1, 5, 107), (2, 2, 64, 112), (1, 2, 3, 961),
    (40, 2, 2, 30), (1, 9, 130, 24), (2, 2, 4, 3), (3, 2, 3, 2), (1, 3, 1, 1), (40, 3, 2, 1),
]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_depthwise_any_size(size, stride, layout):
    B, C, H, W = size
    rng = np.random.default_rng(1000 * W + H)
    if layout == "nhwc":
        C = 3 * C + 1  # quads of channels, with and without a rest
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    w = rng.integers(-127, 128, (C, 1, 3, 3) if layout == "nchw" else (C, 3, 3, 1)).astype(np.int8)
    bias = rng.integers(-10 ** 4, 10 ** 4, C).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(C, 74.0 * 73.0 * 3), 40.0)
    args, rargs = (lay_g, (stride, stride), (1, 1), C), (lay_r, (stride, stride), (1, 1), C)
    w_t, dw = hago.QType(hago.I8), dev(w)
    for adt, za in ((np.uint8, 131), (np.int8, 0), (np.int8, -5)):
        shape = (B, C, H, W) if layout == "nchw" else (B, H, W, C)
        a = (rng.integers(0, 256, shape) if adt == np.uint8 else rng.integers(-128, 128, shape)).astype(adt)
        a_t, da = act_qtype(a, za), dev(a)
        if za == -5:  # a tensor that starts at an odd byte
            buf = torch.zeros(a.size + 1, dtype=torch.int8, device="cuda:0")
            buf[1:] = da.reshape(-1)
            da = buf[1:].reshape(da.shape)
        assert_same(host(hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args)), ref.qconv2d(a, za, w, bias, *rargs), f"raw {size}")
        assert_same(host(hago.qconv2d(da, a_t, dw, w_t, None, *args, hago.I16)), ref.qconv2d(a, za, w, None, *rargs, ref.I16), f"raw 16 {size}")
        for acc, out_u8, z, clip, rounding in ((hago.I32, False, -3, (-128, 127), 0), (hago.I32, True, 10, (10, 255), 1),
                                               (hago.I16, False, 0, (-127, 127), 0)):
            racc = ref.I32 if acc == hago.I32 else ref.I16
            want = ref.qconv2d(a, za, w, bias, *rargs, racc, ref_requant(mult, shift, out_u8, z, clip, rounding))
            got = hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args, acc, gpu_requant(mult, shift, out_u8, z, clip, rounding=rounding))
            assert_same(host(got), want, f"requantized {size} u8={out_u8} acc={acc}")
