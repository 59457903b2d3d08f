"""GPU parity of the convolution that loads both operands straight from memory, both layouts, every tile shape and output
mode, against the oracle: channel counts off the 16-byte chunk, odd numbers of chunks, fewer steps than wavefronts, weights
that stay in registers and that do not, filters that hang over every edge, channel and pixel counts off the tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

CASES = [
    # B C H W O KH KW stride pad
    (1, 16, 4, 5, 3, 1, 1, (1, 1), (0, 0)),        # one chunk
    (2, 17, 7, 9, 33, 3, 3, (1, 1), (1, 1)),       # the second chunk repeats 15 channels
    (3, 31, 6, 5, 64, 1, 1, (2, 2), (0, 0)),
    (2, 48, 9, 9, 70, 3, 3, (2, 2), (1, 1)),       # three chunks a tap: pairs straddle taps
    (1, 64, 13, 11, 65, 5, 5, (1, 1), (2, 2)),
    (5, 40, 7, 7, 45, 3, 3, (1, 1), (1, 1)),
    (2, 18, 6, 8, 5, 3, 3, (1, 1), (4, 4)),        # filters outside the image altogether
    (1, 20, 5, 4, 12, 3, 2, (1, 2), (0, 1)),
    (1, 32, 40, 41, 130, 1, 3, (1, 1), (0, 1)),
    (4, 200, 3, 3, 20, 3, 3, (1, 1), (1, 1)),
    (2, 3, 31, 37, 20, 7, 7, (2, 2), (3, 3)),      # few channels
    (3, 1, 4, 7, 70, 1, 1, (1, 1), (0, 0)),
    (3, 6, 11, 14, 33, 5, 5, (1, 1), (2, 2)),
    (9, 9, 17, 16, 65, 3, 3, (1, 1), (1, 1)),
    (1, 180, 5, 6, 3, 7, 7, (2, 2), (3, 3)),       # a long table
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("shape", [0, 1, 2, 3])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_gathered_convolution(case, shape, layout, gemm_path):
    B, C, H, W, O, KH, KW, stride, pad = case
    if layout == "nhwc" and C >= 16 and shape == 3:  # (three shapes)
        return
    rng = np.random.default_rng(abs(hash(case)) % 2 ** 31)
    w = rng.integers(-127, 128, (O, C, KH, KW)).astype(np.int8)
    bias = rng.integers(-10 ** 5, 10 ** 5, O).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(C * KH * KW)), 40.0)
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    to = (lambda x: x) if layout == "nchw" else (lambda x: np.ascontiguousarray(x.transpose(0, 2, 3, 1)))
    w_t, wl = hago.QType(hago.I8), to(w)
    args, rargs = (lay_g, stride, pad, 1), (lay_r, stride, pad, 1)
    gemm_path(4)
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


@pytest.mark.parametrize("C", [16, 17, 18, 19, 36])
@pytest.mark.parametrize("off_a,off_w", [(1, 0), (0, 2), (3, 1), (2, 3)])
@pytest.mark.parametrize("shape", [0, 1, 2])
def test_operands_at_any_byte(C, off_a, off_w, shape, gemm_path):
    """Rows loaded as aligned dwords: tensors that start and end inside a dword, at the very edges of what is theirs."""
    rng = np.random.default_rng(100 * C + 10 * off_a + off_w)
    a, za = rng.integers(0, 256, (2, 5, 7, C)).astype(np.uint8), 131
    w = rng.integers(-127, 128, (35, 3, 3, C)).astype(np.int8)
    def placed(x, off):
        whole = torch.full((x.size + 32,), 77, dtype=torch.uint8, device="cuda").view(dev(x).dtype)
        at = whole[16 + off: 16 + off + x.size].view(x.shape)
        at.copy_(dev(x))
        return at
    want = ref.qconv2d(a, za, w, None, ref.NHWC, (1, 1), (1, 1), 1)
    gemm_path(4)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, shape)
    try:
        got = hago.qconv2d(placed(a, off_a), act_qtype(a, za), placed(w, off_w), hago.QType(hago.I8), None, hago.NHWC, (1, 1), (1, 1), 1)
        assert_same(host(got), want, f"C={C} off {off_a},{off_w}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)


@pytest.mark.parametrize("layout,C,H,W,KH,stride", [
    ("nchw", 31, 2, 1070000, 5, (1, 4096)),    # image below 2^26 elements, the filter's last tap beyond
    ("nchw", 30, 2, 1070000, 3, (1, 4096)),    # both below
    ("nhwc", 5, 2, 6500003, 5, (1, 4096)),
    ("nhwc", 3, 2, 4000003, 5, (1, 4096)),
])
@pytest.mark.parametrize("path", [0, 4])
def test_filter_taller_than_a_large_image(layout, C, H, W, KH, stride, path, gemm_path):
    """Offsets from a pixel's corner to a filter's last tap, around the 2^26 that the kernel's table holds."""
    to = (lambda x: x) if layout == "nchw" else (lambda x: np.ascontiguousarray(x.transpose(0, 2, 3, 1)))
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    rng = np.random.default_rng(C * KH)
    a = to(rng.integers(0, 256, (1, C, H, W), dtype=np.uint8))
    w = to(rng.integers(-127, 128, (8, C, KH, 5)).astype(np.int8))
    pad = (KH // 2, 2)
    gemm_path(path)
    got = host(hago.qconv2d(dev(a), act_qtype(a, 131), dev(w), hago.QType(hago.I8), None, lay_g, stride, pad))
    assert_same(got, ref.qconv2d(a, 131, w, None, lay_r, stride, pad), f"{layout} {C} x {H} x {W}")
