"""Requantize whose clip is the container's whole range: kernels shift, saturate and pack two results at a time there.
Results on both sides of either limit, the zero points at the ends of their range, shifts on both sides of the ones that
form takes (1 to 19, in the dense layers to 21), and a clip narrower by one, which takes the other form."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

# B C H W O k stride groups layout: one for each kernel with such an epilogue, with remainders of their tiles
LAYERS = {
    "dense_64": (1, 96, 1, 70, 80, 1, 1, 1, "nhwc"),
    "dense_64_long": (1, 400, 1, 70, 80, 1, 1, 1, "nhwc"),
    "dense_128": (1, 64, 1, 2100, 272, 1, 1, 1, "nhwc"),
    "dense_128x256": (1, 144, 1, 300, 272, 1, 1, 1, "nhwc"),
    "dense_192x256": (1, 80, 1, 4100, 2320, 1, 1, 1, "nhwc"),
    "dense_256": (1, 48, 1, 4100, 4112, 1, 1, 1, "nhwc"),
    "pointwise": (2, 24, 9, 15, 33, 1, 1, 1, "nchw"),
    "pointwise_split": (1, 160, 5, 7, 40, 1, 1, 1, "nchw"),
    "conv3x3": (2, 32, 9, 12, 37, 3, 1, 1, "nchw"),
    "direct_nchw": (2, 20, 29, 31, 37, 3, 2, 1, "nchw"),
    "direct_nhwc": (20, 20, 29, 31, 37, 3, 2, 1, "nhwc"),
    "dw_rows": (2, 5, 9, 44, 5, 3, 1, 5, "nchw"),
    "dw_ragged": (2, 5, 9, 67, 5, 3, 1, 5, "nchw"),
    "dw_matrix": (3, 5, 11, 14, 5, 3, 1, 5, "nchw"),
    "dw_matrix_s2": (3, 5, 11, 30, 5, 3, 2, 5, "nchw"),
    "dw_nhwc": (2, 10, 9, 11, 10, 3, 1, 10, "nhwc"),
}
# the dense kernel's tile: which one serves a size is a matter of a fitted rule
TILES = {"dense_64": 4, "dense_64_long": 6, "dense_128": 2, "dense_128x256": 5, "dense_192x256": 1, "dense_256": 0}
FORMS = [  # out_u8, z, clip, shifts
    (False, 0, (-128, 127), (1, 12)), (False, -128, (-128, 127), (6, 9)), (False, 127, (-128, 127), (18, 23)),
    (True, 0, (0, 255), (5, 9)), (True, 255, (0, 255), (0, 4)), (True, 131, (0, 255), (19, 22)),
    (False, 3, (-128, 126), (5, 9)), (True, 7, (1, 255), (5, 9)),
]


@pytest.mark.parametrize("name", LAYERS)
def test_whole_range(name, stream_tile):
    stream_tile(TILES.get(name, -1))
    B, C, H, W, O, k, stride, groups, layout = LAYERS[name]
    rng = np.random.default_rng(sum(map(ord, name)))
    nchw = layout == "nchw"
    for act_u8 in (False, True):
        a = rng.integers(0, 256, (B, C, H, W)).astype(np.uint8) if act_u8 else rng.integers(-128, 128, (B, C, H, W)).astype(np.int8)
        za = 117 if act_u8 else 0
        w = rng.integers(-127, 128, (O, C // groups, k, k)).astype(np.int8)
        bias = rng.integers(-3000, 3000, O).astype(np.int32)
        if not nchw:
            a, w = np.ascontiguousarray(a.transpose(0, 2, 3, 1)), np.ascontiguousarray(w.transpose(0, 2, 3, 1))
        pad, st = (k // 2, k // 2), (stride, stride)
        # one accumulation by the oracle; every form requantizes it
        sums = ref.qconv2d(a, za, w, bias, ref.NCHW if nchw else ref.NHWC, st, pad, groups, ref.I32)
        da, dw, db = dev(a), dev(w), dev(bias)
        for out_u8, z, clip, (s0, s1) in FORMS:
            middling = s0 >= 5 and s1 <= 9
            if middling and groups > 1:  # sums of nine terms: results on both sides of either limit there too
                s0, s1 = s0 - 4, s1 - 4
            mult = rng.integers(2 ** 30, 2 ** 31, O, dtype=np.int64).astype(np.int32)
            shift = rng.integers(s0, s1 + 1, O).astype(np.int32)
            rows = sums.reshape(B, O, -1) if nchw else sums.reshape(-1, O, 1)
            want = ref.requantize(np.ascontiguousarray(rows), ref_requant(mult, shift, out_u8, z, clip)).reshape(sums.shape)
            got = qconv2d(da, act_qtype(a, za), dw, hago.QType(hago.I8), db, hago.NCHW if nchw else hago.NHWC, st, pad, groups,
                          hago.I32, gpu_requant(mult, shift, out_u8, z, clip))
            assert_same(host(got), want, f"{name} u8={act_u8} {out_u8, z, clip, s0, s1}")
            if middling and clip in ((-128, 127), (0, 255)):
                assert (want == clip[0]).any() and (want == clip[1]).any()
                assert groups > 1 or len(np.unique(want)) > 100


@pytest.mark.parametrize("acc", ["I16", "I24"])
@pytest.mark.parametrize("act_u8", [False, True])
def test_whole_range_narrow_accumulator(acc, act_u8):
    """The 3x3 convolution's form for accumulators that wrap: the correction and bias are inside the wrapped sum."""
    rng = np.random.default_rng(5 + act_u8)
    B, C, H, W, O = 2, 64, 9, 12, 37
    a = rng.integers(0, 256, (B, C, H, W)).astype(np.uint8) if act_u8 else rng.integers(-128, 128, (B, C, H, W)).astype(np.int8)
    za = 117 if act_u8 else -5
    w = rng.integers(-127, 128, (O, C, 3, 3)).astype(np.int8)
    bias = rng.integers(-2 ** 23, 2 ** 23, O).astype(np.int32)
    da, dw, db = dev(a), dev(w), dev(bias)
    for out_u8, z, clip, (s0, s1) in FORMS:
        for use_mult in (True, False):
            mult = rng.integers(2 ** 30, 2 ** 31, O, dtype=np.int64).astype(np.int32) if use_mult else None
            shift = rng.integers(s0, s1 + 1, O).astype(np.int32)
            want = ref.qconv2d(a, za, w, bias, ref.NCHW, (1, 1), (1, 1), 1, getattr(ref, acc), ref_requant(mult, shift, out_u8, z, clip))
            rq = hago.Requant(dev(mult), dev(shift), hago.QType(hago.U8 if out_u8 else hago.I8, 8, not out_u8, z), *clip)
            got = hago.qconv2d(da, act_qtype(a, za), dw, hago.QType(hago.I8), db, hago.NCHW, (1, 1), (1, 1), 1, getattr(hago, acc), rq)
            assert_same(host(got), want, f"{acc} u8={act_u8} {out_u8, z, clip, s0, s1} mult={use_mult}")


@pytest.mark.parametrize("acc", ["I16", "I24"])
@pytest.mark.parametrize("tile", [3, 4])   # 128 x 128, which has a form for these, and 64 x 64, which has not
@pytest.mark.parametrize("M, K, N", [(300, 131, 140), (129, 35, 257), (40, 700, 131)])
def test_whole_range_narrow_accumulator_dense(M, K, N, tile, acc, gemm_path):
    """The same in the dense kernel for rows of any size."""
    rng = np.random.default_rng(M + tile)
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, tile)
    try:
        for act_u8 in (False, True):
            a = rng.integers(0, 256, (M, K)).astype(np.uint8) if act_u8 else rng.integers(-128, 128, (M, K)).astype(np.int8)
            za, w = 117 if act_u8 else -5, rng.integers(-127, 128, (N, K)).astype(np.int8)
            bias = rng.integers(-2 ** 23, 2 ** 23, N).astype(np.int32)
            for out_u8, z, clip, (s0, s1) in FORMS:
                mult = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32)
                shift = rng.integers(s0, s1 + 1, N).astype(np.int32)
                want = ref.qdense(a, za, w, bias, getattr(ref, acc), ref_requant(mult, shift, out_u8, z, clip))
                got = hago.qdense(dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), dev(bias), getattr(hago, acc),
                                  gpu_requant(mult, shift, out_u8, z, clip))
                assert_same(host(got), want, f"{M, K, N} u8={act_u8} {out_u8, z, clip, s0, s1}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)


@pytest.mark.parametrize("shape", [(300, 64, 1), (90, 35, 1), (64, 12, 3), (5000, 8, 1)])
@pytest.mark.parametrize("dtype", [np.int32, np.int16])
def test_whole_range_standalone(shape, dtype):
    """The standalone operator on rows whose channels a lane keeps."""
    rng = np.random.default_rng(sum(shape))
    acc = rng.integers(np.iinfo(dtype).min, np.iinfo(dtype).max, shape, endpoint=True).astype(dtype)
    acc[: shape[0] // 2] >>= 9
    for out_u8, z, clip, (s0, s1) in FORMS:
        mult = rng.integers(2 ** 30, 2 ** 31, shape[1], dtype=np.int64).astype(np.int32)
        shift = rng.integers(s0, s1 + 1, shape[1]).astype(np.int32)
        assert_same(host(hago.requantize(dev(acc), gpu_requant(mult, shift, out_u8, z, clip))),
                    ref.requantize(acc, ref_requant(mult, shift, out_u8, z, clip)), f"{shape} {out_u8, z, clip, s0, s1}")
