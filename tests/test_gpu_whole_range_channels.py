"""Whole-range codes with single channels off the saturating form: a shift of 0 or a large one, for which their wavefronts or tiles take the
folded form, and a bias that no folded form takes; every other channel is an ordinary one."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

# B C H W O k stride groups layout: every variant of the kernels by its size
POINTWISE = [
    (1, 160, 5, 27, 40, 1, 1, 1, "nchw"), (2, 24, 9, 15, 70, 1, 1, 1, "nchw"), (3, 30, 7, 7, 40, 1, 1, 1, "nchw"), (3, 40, 12, 14, 70, 1, 1, 1, "nchw"),
    (4, 56, 6, 9, 70, 1, 1, 1, "nchw"), (90, 72, 20, 20, 60, 1, 1, 1, "nchw"), (300, 68, 8, 8, 60, 1, 1, 1, "nchw"), (90, 100, 20, 20, 40, 1, 1, 1, "nchw"),
    (300, 100, 9, 8, 40, 1, 1, 1, "nchw"),
]
DEPTHWISE = [
    (3, 5, 23, 44, 5, 3, 1, 5, "nchw"), (2, 5, 19, 67, 5, 3, 1, 5, "nchw"), (2, 6, 9, 128, 6, 3, 1, 6, "nchw"), (3, 5, 11, 14, 5, 3, 1, 5, "nchw"),
    (3, 5, 11, 7, 5, 3, 1, 5, "nchw"), (3, 5, 21, 40, 5, 3, 1, 5, "nchw"), (3, 5, 11, 30, 5, 3, 2, 5, "nchw"), (2, 10, 9, 11, 10, 3, 1, 10, "nhwc"),
    (2, 10, 9, 11, 10, 3, 2, 10, "nhwc"),
]
DENSE = {  # by the tile that the test forces: every dense kernel with tiles that leave through LDS, and the channel-last convolution
    4: (1, 96, 1, 70, 80, 1, 1, 1, "nhwc"), 6: (1, 400, 1, 70, 80, 1, 1, 1, "nhwc"), 2: (1, 64, 1, 2100, 272, 1, 1, 1, "nhwc"),
    5: (1, 144, 1, 300, 272, 1, 1, 1, "nhwc"), 1: (1, 80, 1, 500, 400, 1, 1, 1, "nhwc"), 0: (1, 48, 1, 500, 400, 1, 1, 1, "nhwc"),
    -1: (4, 128, 28, 28, 128, 3, 1, 1, "nhwc"),
}
LAYERS = [(x, -1) for x in POINTWISE + DEPTHWISE] + [(x, tile) for tile, x in DENSE.items()]


@pytest.mark.parametrize("layer, tile", LAYERS, ids=str)
@pytest.mark.parametrize("act_u8", [False, True])
def test_one_channel_off_the_saturating_form(layer, tile, act_u8, stream_tile):
    stream_tile(tile)
    B, C, H, W, O, k, stride, groups, layout = layer
    rng = np.random.default_rng(sum(layer[:7]) + act_u8)
    nchw = layout == "nchw"
    a = rng.integers(0, 256, (B, C, H, W)).astype(np.uint8) if act_u8 else rng.integers(-128, 128, (B, C, H, W)).astype(np.int8)
    za = 117 if act_u8 else 0
    w = rng.integers(-127, 128, (O, C // groups, k, k)).astype(np.int8)
    if not nchw:
        a, w = np.ascontiguousarray(a.transpose(0, 2, 3, 1)), np.ascontiguousarray(w.transpose(0, 2, 3, 1))
    geo = (stride, stride), (k // 2, k // 2), groups
    sums = ref.qconv2d(a, za, w, None, ref.NCHW if nchw else ref.NHWC, *geo, ref.I32)
    da, dw = dev(a), dev(w)
    channel = (1, O, 1) if nchw else (1, O)
    for odd_shift, odd_bias in ((0, 0), (20, 0), (24, 0), (None, 2 ** 30 + 9), (0, -2 ** 30 - 9)):
        for out_u8, z in ((False, 0), (False, -3), (True, 130)):
            mult = rng.integers(2 ** 30, 2 ** 31, O, dtype=np.int64).astype(np.int32)
            shift = rng.integers(4, 9, O).astype(np.int32) - (3 if groups > 1 else 0)
            bias = rng.integers(-3000, 3000, O).astype(np.int32)
            at = int(rng.integers(0, O))
            bias[at] += odd_bias
            if odd_shift is not None:
                shift[at] = odd_shift
            rows = (sums.reshape(B, O, -1) if nchw else sums.reshape(-1, O)) + bias.reshape(channel)
            want = ref.requantize(np.ascontiguousarray(rows if nchw else rows[:, :, None]), ref_requant(mult, shift, out_u8, z)).reshape(sums.shape)
            got = qconv2d(da, act_qtype(a, za), dw, hago.QType(hago.I8), dev(bias), hago.NCHW if nchw else hago.NHWC, *geo, hago.I32,
                          gpu_requant(mult, shift, out_u8, z))
            assert_same(host(got), want, f"{layer} shift {odd_shift} bias {odd_bias} {out_u8, z}")
