"""GPU parity of the one-launch 3x3 convolution with blocks of 32 and of 64 output channels, and with batches of weight
units that do and do not come out even, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

CASES = [  # B C H W O
    (1, 32, 9, 16, 8), (2, 32, 17, 20, 33), (1, 64, 56, 56, 64), (3, 64, 8, 12, 72), (1, 96, 14, 16, 96), (2, 128, 12, 28, 100),
    (40, 32, 56, 56, 32), (70, 64, 16, 16, 64), (16, 96, 28, 28, 65),
]


@pytest.mark.parametrize("case", CASES)
def test_conv3x3_channel_blocks(case):
    B, C, H, W, O = case
    rng = np.random.default_rng(C * 100 + O)
    w = rng.integers(-127, 128, (O, C, 3, 3)).astype(np.int8)
    bias = rng.integers(-10 ** 4, 10 ** 4, O).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(9 * C)), 40.0)
    args, rargs = (hago.NCHW, (1, 1), (1, 1), 1), (ref.NCHW, (1, 1), (1, 1), 1)
    w_t, dw = hago.QType(hago.I8), dev(w)
    for adt, za in ((np.uint8, 131), (np.int8, 0)):
        a = (rng.integers(0, 256, (B, C, H, W)) if adt == np.uint8 else rng.integers(-128, 128, (B, C, H, W))).astype(adt)
        a_t, da = act_qtype(a, za), dev(a)
        want = ref.qconv2d(a, za, w, bias, *rargs, ref.I32, ref_requant(mult, shift, True, 10, (10, 255), 0))
        got = hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args, hago.I32, gpu_requant(mult, shift, True, 10, (10, 255)))
        assert_same(host(got), want, f"requantized {case}")
        assert_same(host(hago.qconv2d(da, a_t, dw, w_t, dev(bias), *args)), ref.qconv2d(a, za, w, bias, *rargs), f"raw {case}")
