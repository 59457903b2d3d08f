"""GPU parity (bit-exact) of hago_qdense and hago_qconv2d against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen


def rnd_act(rng, shape, dt):
    return rng.integers(0, 256, shape).astype(np.uint8) if dt == np.uint8 else rng.integers(-128, 128, shape).astype(np.int8)


def rnd_w(rng, shape):
    return rng.integers(-127, 128, shape).astype(np.int8)


DENSE_SHAPES = [(1, 1, 1), (3, 4, 5), (64, 128, 256), (77, 53, 100), (130, 129, 65), (200, 24, 144),
                (33, 300, 17), (256, 256, 1024), (5, 7, 0), (300, 64, 2048), (129, 33, 4097)]


@pytest.mark.parametrize("M,N,K", DENSE_SHAPES)
@pytest.mark.parametrize("adt,za", [(np.uint8, 128), (np.uint8, 7), (np.int8, 0), (np.int8, -9)])
def test_qdense_raw_int32(M, N, K, adt, za):
    rng = np.random.default_rng(abs(hash((M, N, K, za))) % 2 ** 31)
    a, w = rnd_act(rng, (M, K), adt), rnd_w(rng, (N, K))
    bias = rng.integers(-10 ** 6, 10 ** 6, N).astype(np.int32)
    want = ref.qdense(a, za, w, bias)
    got = hago.qdense(dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), dev(bias))
    assert_same(host(got), want, f"qdense raw {M}x{N}x{K}")


@pytest.mark.parametrize("M,N,K", [(64, 128, 256), (77, 53, 100), (130, 132, 320), (31, 24, 144)])
def test_qdense_requant_and_acc16(M, N, K):
    rng = np.random.default_rng(M * 7 + N)
    a, w = rnd_act(rng, (M, K), np.uint8), rnd_w(rng, (N, K))
    mult, shift = datagen.requant_params(rng, np.full(N, 74.0 * 73.0 * np.sqrt(max(K, 1))), 40.0)
    for out_u8, z_out, clip in ((False, 0, (-128, 127)), (True, 10, (10, 255)), (False, 1, (-8, 7))):
        want = ref.qdense(a, 131, w, None, ref.I32, ref_requant(mult, shift, out_u8, z_out, clip))
        got = hago.qdense(dev(a), act_qtype(a, 131), dev(w), hago.QType(hago.I8), None, hago.I32,
                          gpu_requant(mult, shift, out_u8, z_out, clip, bits=4 if clip == (-8, 7) else 8))
        assert_same(host(got), want, f"qdense rq {M}x{N}x{K} u8={out_u8}")
        sat = np.mean((want == clip[0]) | (want == clip[1]))
        assert sat < 0.9
    # per-tensor parameters
    want = ref.qdense(a, 131, w, None, ref.I32, ref_requant(mult[:1], shift[:1]))
    got = hago.qdense(dev(a), act_qtype(a, 131), dev(w), hago.QType(hago.I8), None, hago.I32,
                      gpu_requant(mult[:1], shift[:1]))
    assert_same(host(got), want, "per-tensor")
    # int16 accumulation: raw and requantized; 8-bit operands wrap constantly here
    a8 = rnd_act(rng, (M, K), np.int8)
    want = ref.qdense(a8, 3, w, None, ref.I16)
    got = hago.qdense(dev(a8), act_qtype(a8, 3), dev(w), hago.QType(hago.I8), None, hago.I16)
    assert_same(host(got), want, "acc16 raw")
    m16, s16 = datagen.requant_params(rng, np.full(N, 19000.0), 40.0)
    want = ref.qdense(a8, 3, w, None, ref.I16, ref_requant(m16, s16))
    got = hago.qdense(dev(a8), act_qtype(a8, 3), dev(w), hago.QType(hago.I8), None, hago.I16, gpu_requant(m16, s16))
    assert_same(host(got), want, "acc16 requant")


# 256 x 256, 192 x 256, 128 x 128 (2 and 3), 64 x 64, 128 x 256, 64 x 64 with 128-byte stages
@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("K", [448, 400, 64, 16])  # whole 64-byte stages / a 16-byte tail / one stage
@pytest.mark.parametrize("adt,za", [(np.uint8, 121), (np.uint8, 128), (np.int8, -4)])
def test_qdense_every_tile_shape(tile, K, adt, za, stream_tile):
    """Each dense tile shape of the LDS-DMA kernel on a shape with several tiles and ragged edges
    in both directions, requantized (staged and plain epilogues) and raw."""
    stream_tile(tile)
    M, N = 600, 528
    rng = np.random.default_rng(tile * 1000 + K + za)
    a, w = rnd_act(rng, (M, K), adt), rnd_w(rng, (N, K))
    bias = rng.integers(-10 ** 5, 10 ** 5, N).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(N, 74.0 * 73.0 * np.sqrt(K)), 40.0)
    want = ref.qdense(a, za, w, bias, ref.I32, ref_requant(mult, shift))
    got = hago.qdense(dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), dev(bias), hago.I32,
                      gpu_requant(mult, shift))
    assert_same(host(got), want, f"tile {tile} K={K} requantized")
    assert np.mean((want == -128) | (want == 127)) < 0.5
    want = ref.qdense(a, za, w, bias)
    got = hago.qdense(dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), dev(bias))
    assert_same(host(got), want, f"tile {tile} K={K} raw")


def test_qdense_config1_both_variants():
    for variant in ("as_specified", "discriminating"):
        c = datagen.config1(variant=variant)
        want = ref.qdense(c["a"], c["z_a"], c["w"], None, ref.I32, ref_requant(c["mult"], c["shift"]))
        got = hago.qdense(dev(c["a"]), act_qtype(c["a"], c["z_a"]), dev(c["w"]), hago.QType(hago.I8), None,
                          hago.I32, gpu_requant(c["mult"], c["shift"]))
        assert_same(host(got), want, f"config 1 {variant}")
        if variant == "discriminating":
            assert np.mean(np.abs(want.astype(np.int32)) >= 127) < 0.5


@pytest.mark.parametrize("idx", [0, 1, 2, 3])
def test_qdense_config5_full_size(idx):
    """Every element of every layer of the benchmark stack, in the launch configuration bench.py times."""
    import os
    c = datagen.config5_layer(idx)
    got = host(hago.qdense(dev(c["a"]), act_qtype(c["a"], c["z_a"]), dev(c["w"]), hago.QType(hago.I8),
                           dev(c["bias"]), hago.I32, gpu_requant(c["mult"], c["shift"])))
    want = ref.qdense_threaded(c["a"], c["z_a"], c["w"], c["bias"], ref.I32, ref_requant(c["mult"], c["shift"]),
                               threads=min(16, os.cpu_count() or 1))
    assert_same(got, want, f"config 5 layer {idx}")
    sat = np.mean(np.abs(want.astype(np.int32)) >= 127)
    assert sat < 0.05, sat
    assert want.std() > 10


def _extreme_terms(rng, N):
    """Bias and shift vectors that put channels on both sides of every switch of the fused epilogue:
    |bias| around 2^30 (where the folded 64-bit constant stops being usable), INT32 extremes (the
    accumulator wraps), shifts 0 and 31 next to ordinary ones."""
    bias = rng.integers(-10 ** 5, 10 ** 5, N).astype(np.int64)
    shift = rng.integers(6, 14, N).astype(np.int32)
    special = [2 ** 30 - 7, 2 ** 30 + 7, -(2 ** 30) + 7, -(2 ** 30) - 7, 2 ** 31 - 1, -(2 ** 31), 2 ** 30, -(2 ** 30)]
    for k, b in enumerate(special):
        for base in (3, 70, 200, 333, N - 40):      # spread over every 32-channel block a tile may hold
            if 0 <= base + 5 * k < N:
                bias[base + 5 * k] = b
    for base in (1, 64, 129, 250, 300, N - 9):
        if 0 <= base < N - 2:
            shift[base], shift[base + 2] = 0, 31
    return bias.astype(np.int32), shift


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("out_u8,z_out", [(False, 0), (True, 131), (False, -9)])
def test_qdense_epilogue_switches_every_tile(tile, out_u8, z_out, stream_tile):
    """The streaming kernel's fused epilogue picks, per tile, between the folded arithmetic and the
    general one (a shift of 0, a bias term near 2^30); both kinds of channel inside one staged tile,
    for every tile shape, multi-tile and ragged, against the oracle's wrapping arithmetic."""
    stream_tile(tile)
    M, N, K = 520, 400, 448
    rng = np.random.default_rng(4000 + tile * 10 + z_out)
    a, w = rnd_act(rng, (M, K), np.uint8), rnd_w(rng, (N, K))
    bias, shift = _extreme_terms(rng, N)
    mult = rng.integers(2 ** 30, 2 ** 31, N).astype(np.int32)
    want = ref.qdense(a, 121, w, bias, ref.I32, ref_requant(mult, shift, out_u8, z_out))
    got = hago.qdense(dev(a), act_qtype(a, 121), dev(w), hago.QType(hago.I8), dev(bias), hago.I32,
                      gpu_requant(mult, shift, out_u8, z_out))
    assert_same(host(got), want, f"tile {tile} extreme terms")
    assert len(np.unique(want)) > 100
    # a tile whose channels are all ordinary next to tiles that are not: ordinary terms only in the first 256
    bias2, shift2 = bias.copy(), shift.copy()
    bias2[:256] = rng.integers(-10 ** 5, 10 ** 5, 256)
    shift2[:256] = rng.integers(6, 14, 256)
    want = ref.qdense(a, 121, w, bias2, ref.I32, ref_requant(mult, shift2, out_u8, z_out))
    got = hago.qdense(dev(a), act_qtype(a, 121), dev(w), hago.QType(hago.I8), dev(bias2), hago.I32,
                      gpu_requant(mult, shift2, out_u8, z_out))
    assert_same(host(got), want, f"tile {tile} mixed tiles")
    # raw accumulators with the same biases: the int32 wrap of acc + bias
    want = ref.qdense(a, 121, w, bias)
    assert_same(host(hago.qdense(dev(a), act_qtype(a, 121), dev(w), hago.QType(hago.I8), dev(bias))), want, "raw wrap")


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("O", [72, 200])
def test_qconv2d_epilogue_switches(layout, O):
    """The same switches through the 3x3 implicit GEMM on the workspace path (several tiles, ragged)."""
    B, C, H, W = 2, 32, 19, 24
    rng = np.random.default_rng(5100 + O)
    a, w = rnd_act(rng, (B, C, H, W), np.uint8), rnd_w(rng, (O, C, 3, 3))
    bias, shift = _extreme_terms(rng, O)
    mult = rng.integers(2 ** 30, 2 ** 31, O).astype(np.int32)
    lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
    ah = a if layout == "nchw" else np.ascontiguousarray(a.transpose(0, 2, 3, 1))
    wh = w if layout == "nchw" else np.ascontiguousarray(w.transpose(0, 2, 3, 1))
    need = hago.qconv2d_workspace_bytes(ah.shape, wh.shape, lay_g, (1, 1), (1, 1))
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    for out_u8, z_out in ((False, 0), (True, 131)):
        want = ref.qconv2d(ah, 128, wh, bias, lay_r, (1, 1), (1, 1), 1, ref.I32, ref_requant(mult, shift, out_u8, z_out))
        got = hago.qconv2d(dev(ah), act_qtype(ah, 128), dev(wh), hago.QType(hago.I8), dev(bias), lay_g, (1, 1), (1, 1), 1,
                           hago.I32, gpu_requant(mult, shift, out_u8, z_out), workspace=ws)
        assert_same(host(got), want, f"conv extreme terms {layout} u8={out_u8}")
    # the weights part of the workspace is still valid: skip its rewrite
    want = ref.qconv2d(ah, 128, wh, bias, lay_r, (1, 1), (1, 1), 1)
    got = hago.qconv2d(dev(ah), act_qtype(ah, 128), dev(wh), hago.QType(hago.I8), dev(bias), lay_g, (1, 1), (1, 1), 1,
                       hago.I32, None, flags=hago.WS_WEIGHTS_READY, workspace=ws)
    assert_same(host(got), want, f"conv raw, weights kept {layout}")


def test_qdense_long_reduction_takes_the_general_epilogue():
    """K > 65536: |acc| may exceed 2^30, so the folded constant is not used; int8 activations at their
    extremes make the accumulator wrap."""
    M, N, K = 40, 48, 66048
    rng = np.random.default_rng(66)
    a = np.where(rng.random((M, K)) < 0.9, 127, -128).astype(np.int8)
    w = np.where(rng.random((N, K)) < 0.9, 127, -127).astype(np.int8)
    bias = rng.integers(-10 ** 6, 10 ** 6, N).astype(np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, N).astype(np.int32)
    shift = rng.integers(18, 24, N).astype(np.int32)
    want = ref.qdense(a, -3, w, bias, ref.I32, ref_requant(mult, shift))
    got = hago.qdense(dev(a), act_qtype(a, -3), dev(w), hago.QType(hago.I8), dev(bias), hago.I32, gpu_requant(mult, shift))
    assert_same(host(got), want, "K = 66048")
    assert np.abs(ref.qdense(a, -3, w, bias).astype(np.int64)).max() > 2 ** 29


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5, 6])
def test_general_kernel_every_tile_dense(tile, gemm_path):
    """The register-staged kernel (what unaligned or oversized operands get) forced on an aligned
    shape, one tile shape at a time."""
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, tile)
    try:
        M, N, K = 300, 272, 208
        rng = np.random.default_rng(900 + tile)
        a, w = rnd_act(rng, (M, K), np.uint8), rnd_w(rng, (N, K))
        bias = rng.integers(-10 ** 5, 10 ** 5, N).astype(np.int32)
        mult, shift = datagen.requant_params(rng, np.full(N, 74.0 * 73.0 * np.sqrt(K)), 40.0)
        want = ref.qdense(a, 119, w, bias, ref.I32, ref_requant(mult, shift))
        got = hago.qdense(dev(a), act_qtype(a, 119), dev(w), hago.QType(hago.I8), dev(bias), hago.I32, gpu_requant(mult, shift))
        assert_same(host(got), want, f"general kernel tile {tile}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_general_kernel_every_tile_conv(tile, layout, gemm_path):
    """The general kernel's implicit-GEMM loaders for both layouts, one tile shape at a time (shapes a
    layout cannot instantiate fall back to 128 x 128), with a workspace present that must stay unused."""
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, tile)
    try:
        B, C, H, W, O = 2, 48, 13, 20, 136
        rng = np.random.default_rng(950 + tile)
        a, w = rnd_act(rng, (B, C, H, W), np.uint8), rnd_w(rng, (O, C, 3, 3))
        bias = rng.integers(-10 ** 5, 10 ** 5, O).astype(np.int32)
        mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(9 * C)), 40.0)
        lay_g, lay_r = (hago.NCHW, ref.NCHW) if layout == "nchw" else (hago.NHWC, ref.NHWC)
        ah = a if layout == "nchw" else np.ascontiguousarray(a.transpose(0, 2, 3, 1))
        wh = w if layout == "nchw" else np.ascontiguousarray(w.transpose(0, 2, 3, 1))
        ws = torch.full((hago.qconv2d_workspace_bytes(ah.shape, wh.shape, lay_g, (1, 1), (1, 1)),), 0x77,
                        dtype=torch.uint8, device=DEV)
        for acc_g, acc_r, rq in ((hago.I32, ref.I32, True), (hago.I32, ref.I32, False), (hago.I16, ref.I16, False)):
            want = ref.qconv2d(ah, 125, wh, bias, lay_r, (1, 1), (1, 1), 1, acc_r, ref_requant(mult, shift) if rq else None)
            got = hago.qconv2d(dev(ah), act_qtype(ah, 125), dev(wh), hago.QType(hago.I8), dev(bias), lay_g, (1, 1), (1, 1), 1,
                               acc_g, gpu_requant(mult, shift) if rq else None, workspace=ws)
            assert_same(host(got), want, f"general conv tile {tile} {layout} rq={rq}")
        assert bool((ws == 0x77).all())
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)


CONV_CASES = [
    # B C H W O KH KW stride pad
    (1, 3, 5, 6, 4, 3, 3, (1, 1), (1, 1)),
    (2, 4, 7, 5, 6, 3, 3, (2, 2), (1, 1)),
    (1, 2, 6, 6, 3, 1, 1, (1, 1), (0, 0)),
    (1, 3, 8, 7, 2, 3, 2, (1, 2), (0, 1)),
    (1, 2, 4, 4, 2, 5, 5, (1, 1), (2, 2)),
    (2, 16, 12, 12, 40, 3, 3, (1, 1), (1, 1)),
    (3, 32, 9, 11, 70, 3, 3, (1, 1), (1, 1)),
    (1, 64, 14, 14, 130, 1, 1, (1, 1), (0, 0)),
    (2, 48, 8, 8, 24, 1, 1, (1, 1), (0, 0)),
    (1, 3, 33, 33, 16, 7, 7, (2, 2), (3, 3)),
    # stride 1 with channel counts that are multiples of 32; ragged tiles in pixels and channels
    (2, 64, 19, 37, 72, 3, 3, (1, 1), (1, 1)),
    (1, 96, 10, 33, 64, 5, 5, (1, 1), (2, 2)),
    (1, 128, 9, 40, 130, 3, 3, (1, 1), (0, 0)),
    (2, 32, 17, 30, 8, 1, 3, (1, 1), (0, 1)),
    # NCHW widths that are multiples of 4 (the transposing operand rewrite): channel counts off the
    # 16- and 64-channel groups, padding that differs between the axes or is absent on one
    (1, 80, 6, 8, 20, 3, 3, (1, 1), (1, 1)),
    (2, 3, 5, 8, 4, 3, 5, (1, 1), (1, 2)),
    (1, 20, 7, 12, 9, 3, 1, (1, 1), (1, 0)),
    (3, 70, 4, 4, 5, 3, 3, (1, 1), (1, 1)),
]


@pytest.mark.parametrize("case", CONV_CASES)
@pytest.mark.parametrize("adt,za", [(np.uint8, 128), (np.uint8, 3), (np.int8, 0), (np.int8, -5)])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_qconv2d_raw(case, adt, za, layout, conv_entry):
    B, C, H, W, O, KH, KW, stride, pad = case
    rng = np.random.default_rng(abs(hash((case, za))) % 2 ** 31)
    a = rnd_act(rng, (B, C, H, W), adt)
    w = rnd_w(rng, (O, C, KH, KW))
    bias = rng.integers(-5000, 5000, O).astype(np.int32)
    want = ref.qconv2d(a, za, w, bias, ref.NCHW, stride, pad, 1)
    if layout == "nchw":
        got = host(qconv2d(dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), dev(bias), hago.NCHW, stride, pad))
    else:
        got = host(qconv2d(dev(a.transpose(0, 2, 3, 1)), act_qtype(a, za), dev(w.transpose(0, 2, 3, 1)),
                                hago.QType(hago.I8), dev(bias), hago.NHWC, stride, pad)).transpose(0, 3, 1, 2)
    assert_same(np.ascontiguousarray(got), want, f"qconv2d {layout} {case}")


@pytest.mark.parametrize("case", [c for c in CONV_CASES if c[1] % 32 == 0 and c[7] == (1, 1) and c[5] * c[6] > 1])
def test_qconv2d_output_modes(case, conv_entry):
    """Requantized (int8 and uint8 with a zero point), raw int16 and requantized int16-accumulation
    outputs of the implicit-GEMM convolution on multi-tile shapes."""
    B, C, H, W, O, KH, KW, stride, pad = case
    rng = np.random.default_rng(B * 100 + C + W)
    a = rnd_act(rng, (B, C, H, W), np.uint8)
    w = rnd_w(rng, (O, C, KH, KW))
    bias = rng.integers(-5000, 5000, O).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(C * KH * KW)), 40.0)
    for out_u8, z_out, clip in ((False, 0, (-128, 127)), (True, 7, (7, 255))):
        want = ref.qconv2d(a, 99, w, bias, ref.NCHW, stride, pad, 1, ref.I32,
                           ref_requant(mult, shift, out_u8, z_out, clip))
        got = qconv2d(dev(a), act_qtype(a, 99), dev(w), hago.QType(hago.I8), dev(bias), hago.NCHW,
                           stride, pad, 1, hago.I32, gpu_requant(mult, shift, out_u8, z_out, clip))
        assert_same(host(got), want, f"conv requantized u8={out_u8}")
        assert np.mean((want == clip[0]) | (want == clip[1])) < 0.6
    want = ref.qconv2d(a, 99, w, bias, ref.NCHW, stride, pad, 1, ref.I16)
    got = qconv2d(dev(a), act_qtype(a, 99), dev(w), hago.QType(hago.I8), dev(bias), hago.NCHW, stride,
                       pad, 1, hago.I16)
    assert_same(host(got), want, "conv raw int16")
    m16, s16 = datagen.requant_params(rng, np.full(O, 19000.0), 40.0)
    want = ref.qconv2d(a, 99, w, bias, ref.NCHW, stride, pad, 1, ref.I16, ref_requant(m16, s16))
    got = qconv2d(dev(a), act_qtype(a, 99), dev(w), hago.QType(hago.I8), dev(bias), hago.NCHW, stride,
                       pad, 1, hago.I16, gpu_requant(m16, s16))
    assert_same(host(got), want, "conv int16 accumulation requantized")


POINTWISE_CASES = [
    # B C H W O: 1x1 stride-1 unpadded NCHW convolutions with C % 16 == 0 and H*W % 4 == 0 (the
    # direct kernel): partial pixel tiles, one / two / four channel tiles per wavefront
    (2, 16, 6, 6, 5), (1, 48, 5, 8, 33), (3, 32, 10, 10, 70), (1, 160, 4, 7, 128), (2, 208, 16, 12, 24),
    # up to 32 output channels: 128 pixels per wavefront, 16-byte stores when H*W % 16 == 0
    (1, 144, 28, 28, 24), (2, 32, 9, 16, 32), (1, 16, 2, 2, 1), (1, 336, 13, 12, 17),
    # few input channels, many output channels (the expansion layers): blocks of 32 output
    # channels per workgroup row; channel counts that are multiples of 4 but not of 16
    (2, 24, 12, 12, 144), (1, 16, 8, 8, 96), (1, 36, 6, 6, 40), (2, 64, 4, 4, 384), (1, 8, 6, 6, 5),
    (1, 4, 2, 2, 70), (1, 20, 14, 14, 33),
]


@pytest.mark.parametrize("case", POINTWISE_CASES)
@pytest.mark.parametrize("adt,za", [(np.uint8, 7), (np.int8, -3)])
def test_pointwise_nchw_all_output_modes(case, adt, za, conv_entry):
    B, C, H, W, O = case
    rng = np.random.default_rng(abs(hash((case, za))) % 2 ** 31)
    a = rnd_act(rng, (B, C, H, W), adt)
    w = rnd_w(rng, (O, C, 1, 1))
    bias = rng.integers(-5000, 5000, O).astype(np.int32)
    args = (hago.NCHW, (1, 1), (0, 0), 1)
    rargs = (ref.NCHW, (1, 1), (0, 0), 1)
    a_t, w_t = act_qtype(a, za), hago.QType(hago.I8)
    want = ref.qconv2d(a, za, w, bias, *rargs)
    assert_same(host(qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args)), want, f"pointwise raw {case}")
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(C)), 40.0)
    for out_u8, z_out, clip in ((False, 0, (-128, 127)), (True, 9, (9, 255))):
        want = ref.qconv2d(a, za, w, bias, *rargs, ref.I32, ref_requant(mult, shift, out_u8, z_out, clip))
        got = qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I32,
                           gpu_requant(mult, shift, out_u8, z_out, clip))
        assert_same(host(got), want, f"pointwise rq {case} u8={out_u8}")
        assert np.mean((want == clip[0]) | (want == clip[1])) < 0.9
    want = ref.qconv2d(a, za, w, bias, *rargs, ref.I16)
    assert_same(host(qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I16)), want, f"pointwise acc16 {case}")
    m16, s16 = datagen.requant_params(rng, np.full(O, 19000.0), 40.0)
    want = ref.qconv2d(a, za, w, bias, *rargs, ref.I16, ref_requant(m16[:1], s16[:1]))
    got = qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I16, gpu_requant(m16[:1], s16[:1]))
    assert_same(host(got), want, f"pointwise acc16 requant per-tensor {case}")


@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("out_u8,z_out", [(False, -7), (True, 131)])
def test_pointwise_requant_constant_ranges(big, out_u8, z_out):
    """The 128-pixel pointwise kernel folds bias term, rounding term and output zero point into one 64-bit
    constant per channel when every channel's constants are small enough (big=False: at the bounds) and
    takes the general form otherwise (big=True: beyond them)."""
    B, C, H, W, O = 2, 48, 12, 12, 24
    rng = np.random.default_rng(500 + z_out + big)
    a = rnd_act(rng, (B, C, H, W), np.uint8)
    w = rnd_w(rng, (O, C, 1, 1))
    bias = rng.integers(-5000, 5000, O).astype(np.int64)
    shift = rng.integers(5, 12, O).astype(np.int32)
    shift[:4] = [0, 1, 19, 19]
    bias[4], bias[5] = 2 ** 30 - 2 ** 22, -(2 ** 30) + 2 ** 22
    if big:
        shift[6:9] = [20, 31, 25]
        bias[9], bias[10], bias[11] = 2 ** 31 - 1, -(2 ** 31), 2 ** 30 + 2 ** 23
    bias = bias.astype(np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, size=O).astype(np.int32)
    a_t, w_t = act_qtype(a, 121), hago.QType(hago.I8)
    want = ref.qconv2d(a, 121, w, bias, ref.NCHW, (1, 1), (0, 0), 1, ref.I32, ref_requant(mult, shift, out_u8, z_out))
    got = qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), hago.NCHW, (1, 1), (0, 0), 1, hago.I32,
                       gpu_requant(mult, shift, out_u8, z_out))
    assert_same(host(got), want, "pointwise requant ranges")
    assert len(np.unique(want)) > 50


def test_qconv2d_config2_full_size(conv_entry):
    for z_a in (0, 128):
        c = datagen.config2(z_a=z_a)
        rq = ref_requant(c["mult"], c["shift"], True, 0, (0, 255))
        want = ref.qconv2d(c["a"], z_a, c["w"], None, ref.NCHW, (1, 1), (1, 1), 1, ref.I32, rq)
        got = qconv2d(dev(c["a"]), act_qtype(c["a"], z_a), dev(c["w"]), hago.QType(hago.I8), None, hago.NCHW,
                           (1, 1), (1, 1), 1, hago.I32, gpu_requant(c["mult"], c["shift"], True, 0, (0, 255)))
        assert_same(host(got), want, f"config 2 z_a={z_a}")
        assert 0.2 < np.mean(want == 0) < 0.8       # the ReLU clip removes about half
        assert np.mean(want == 255) < 0.05


def test_qconv2d_config3_int16_accumulation_full_size(conv_entry):
    for adversarial in (False, True):
        c = datagen.config3(adversarial=adversarial)
        want = ref.qconv2d(c["a"], 0, c["w"], None, ref.NCHW, (1, 1), (1, 1), 1, ref.I16)
        a_t = hago.QType(hago.I8, 4, False, 0)
        w_t = hago.QType(hago.I8, 4, True, 0)
        got = qconv2d(dev(c["a"]), a_t, dev(c["w"]), w_t, None, hago.NCHW, (1, 1), (1, 1), 1, hago.I16)
        assert_same(host(got), want, f"config 3 adversarial={adversarial}")
        if adversarial:
            assert want[0, 0, 5, 5] == -10112      # 1152 * 15 * 7 = 120960 wraps
        else:
            w32 = ref.qconv2d(c["a"][:1], 0, c["w"], None, ref.NCHW, (1, 1), (1, 1), 1, ref.I32)
            assert np.array_equal(w32, want[:1].astype(np.int32))  # random data does not reach the wrap
        # the declared 4-bit ranges do not prove safety for K = 1152
        with pytest.raises(hago.HagoError) as e:
            qconv2d(dev(c["a"]), a_t, dev(c["w"]), w_t, None, hago.NCHW, (1, 1), (1, 1), 1, hago.I16,
                         flags=hago.STRICT_ACC16)
        assert e.value.code == 6


DIRECT3X3_CASES = [
    # B C H W O : NCHW 3x3 stride 1 pad 1 without a workspace -> the one-launch kernel
    (1, 32, 5, 8, 7),         # one partial tile, fewer than 32 output channels
    (2, 64, 9, 56, 64),       # tiles of two rows, the last one a single row
    (1, 64, 56, 56, 64),      # config 2's geometry
    (3, 128, 28, 28, 128),    # config 3's geometry: two blocks of output channels
    (2, 96, 7, 60, 65),       # H * W not a multiple of 16: byte stores; a second block with one channel
    (1, 32, 3, 128, 130),     # one row per tile, the widest image the kernel takes
    (2, 32, 40, 4, 33),       # narrow images: 32 rows per tile
    (1, 128, 16, 16, 24),
]


@pytest.mark.parametrize("case", DIRECT3X3_CASES)
@pytest.mark.parametrize("adt,za", [(np.uint8, 128), (np.uint8, 3), (np.int8, -5)])
def test_qconv2d_one_launch_3x3(case, adt, za):
    """hago_qconv2d without scratch on the geometries its one-launch kernel takes: every output mode."""
    B, C, H, W, O = case
    rng = np.random.default_rng(abs(hash(case)) % 2 ** 31 + za)
    a, w = rnd_act(rng, (B, C, H, W), adt), rnd_w(rng, (O, C, 3, 3))
    bias = rng.integers(-10 ** 5, 10 ** 5, O).astype(np.int32)
    a_t, w_t = act_qtype(a, za), hago.QType(hago.I8)
    args = (hago.NCHW, (1, 1), (1, 1), 1)
    rargs = (ref.NCHW, (1, 1), (1, 1), 1)
    assert_same(host(hago.qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args)), ref.qconv2d(a, za, w, bias, *rargs), f"raw {case}")
    assert_same(host(hago.qconv2d(dev(a), a_t, dev(w), w_t, None, *args, hago.I16)), ref.qconv2d(a, za, w, None, *rargs, ref.I16),
                f"raw int16 {case}")
    assert_same(host(hago.qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I24)), ref.qconv2d(a, za, w, bias, *rargs, ref.I24),
                f"24-bit {case}")
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(9 * C)), 40.0)
    shift[0] = 0
    for out_u8, z_out, clip, rounding in ((False, 0, (-128, 127), 0), (True, 10, (10, 255), 1), (False, -3, (-8, 7), 0)):
        want = ref.qconv2d(a, za, w, bias, *rargs, ref.I32, ref_requant(mult, shift, out_u8, z_out, clip, rounding))
        got = hago.qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I32,
                           gpu_requant(mult, shift, out_u8, z_out, clip, bits=4 if clip == (-8, 7) else 8, rounding=rounding))
        assert_same(host(got), want, f"requantized {case} u8={out_u8}")
    assert np.mean((want == -8) | (want == 7)) < 0.95
    # unaligned output pointer: the 16-byte stores give way to single ones
    buf = torch.empty(B * O * H * W + 1, dtype=torch.int8, device=DEV)
    out = buf[1:].view(B, O, H, W)
    want = ref.qconv2d(a, za, w, bias, *rargs, ref.I32, ref_requant(mult, shift))
    hago.qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I32, gpu_requant(mult, shift), out=out)
    assert_same(host(out), want, f"unaligned output {case}")


def test_qconv2d_one_launch_3x3_small_then_large_lds():
    """One instantiation of the one-launch kernel serves geometries with different LDS sizes (the size depends
    on the image width and rows per tile): a call that needs little LDS followed by calls that need more than
    the 64 KB default limit."""
    rng = np.random.default_rng(99)
    for B, C, H, W, O in ((1, 64, 4, 8, 16), (1, 64, 56, 56, 64), (1, 64, 8, 120, 64), (70, 64, 8, 8, 64), (130, 64, 16, 60, 64)):
        a, w = rnd_act(rng, (B, C, H, W), np.uint8), rnd_w(rng, (O, C, 3, 3))
        want = ref.qconv2d(a, 128, w, None, ref.NCHW, (1, 1), (1, 1), 1)
        got = hago.qconv2d(dev(a), act_qtype(a, 128), dev(w), hago.QType(hago.I8), None, hago.NCHW, (1, 1), (1, 1), 1)
        assert_same(host(got), want, f"raw {(B, C, H, W, O)}")


@pytest.mark.parametrize("O", [128, 100])
def test_qconv2d_many_pixels_128_channels(O, conv_entry):
    """3x3 convolution with 128 input channels over more than 2^15 output pixels (the 256-pixel
    implicit-GEMM tiles, full and ragged in the channels), all three output modes."""
    B, C, H, W = 44, 128, 28, 28
    rng = np.random.default_rng(31 + O)
    a = rnd_act(rng, (B, C, H, W), np.uint8)
    w = rnd_w(rng, (O, C, 3, 3))
    bias = rng.integers(-5000, 5000, O).astype(np.int32)
    a_t, w_t = act_qtype(a, 119), hago.QType(hago.I8)
    args = (hago.NCHW, (1, 1), (1, 1), 1)
    rargs = (ref.NCHW, (1, 1), (1, 1), 1)
    want = ref.qconv2d(a, 119, w, bias, *rargs)
    assert_same(host(qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args)), want, "raw int32")
    mult, shift = datagen.requant_params(rng, np.full(O, 74.0 * 73.0 * np.sqrt(9 * C)), 40.0)
    want = ref.qconv2d(a, 119, w, bias, *rargs, ref.I32, ref_requant(mult, shift))
    got = qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I32, gpu_requant(mult, shift))
    assert_same(host(got), want, "requantized")
    assert len(np.unique(want)) > 100
    want = ref.qconv2d(a, 119, w, bias, *rargs, ref.I16)
    assert_same(host(qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), *args, hago.I16)), want, "raw int16")


def test_config4_mobilenet_block_full_size(conv_entry):
    c = datagen.config4()
    a_t = hago.QType(hago.I8, 8, True, 0)
    w_t = hago.QType(hago.I8)
    rq_dw = ref_requant(c["mult_dw"], c["shift_dw"])
    want_dw = ref.qconv2d(c["a"], 0, c["w_dw"], None, ref.NCHW, (1, 1), (1, 1), 144, ref.I32, rq_dw)
    got_dw = qconv2d(dev(c["a"]), a_t, dev(c["w_dw"]), w_t, None, hago.NCHW, (1, 1), (1, 1), 144, hago.I32,
                          gpu_requant(c["mult_dw"], c["shift_dw"]))
    assert_same(host(got_dw), want_dw, "config 4 depthwise")
    assert np.mean(np.abs(want_dw.astype(np.int32)) >= 127) < 0.05
    rq_pw = ref_requant(c["mult_pw"], c["shift_pw"])
    want_pw = ref.qconv2d(want_dw, 0, c["w_pw"], None, ref.NCHW, (1, 1), (0, 0), 1, ref.I32, rq_pw)
    got_pw = qconv2d(got_dw, a_t, dev(c["w_pw"]), w_t, None, hago.NCHW, (1, 1), (0, 0), 1, hago.I32,
                          gpu_requant(c["mult_pw"], c["shift_pw"]))
    assert_same(host(got_pw), want_pw, "config 4 pointwise")
    assert np.mean(np.abs(want_pw.astype(np.int32)) >= 127) < 0.05


DW_CASES = [
    # B C H W KH KW stride pad
    (2, 5, 6, 7, 3, 3, (1, 1), (1, 1)),
    (1, 4, 9, 9, 3, 3, (2, 2), (0, 0)),
    (2, 3, 56, 56, 3, 3, (1, 1), (1, 1)),
    (1, 2, 150, 20, 3, 3, (1, 1), (1, 1)),     # more rows than one band
    (1, 3, 17, 31, 3, 3, (1, 1), (1, 1)),      # width not a multiple of 4
    (1, 6, 12, 12, 5, 5, (1, 1), (2, 2)),
    (1, 2, 8, 300, 3, 3, (1, 1), (1, 1)),
    # stride 2, pad 1 (the downsampling layers): dword-merged stores (W % 8 == 0) and 16-bit stores,
    # odd heights, more output rows than one band, widths the register kernel does not take
    (2, 6, 56, 56, 3, 3, (2, 2), (1, 1)),
    (1, 3, 28, 28, 3, 3, (2, 2), (1, 1)),
    (1, 2, 150, 20, 3, 3, (2, 2), (1, 1)),
    (2, 5, 9, 16, 3, 3, (2, 2), (1, 1)),
    (1, 4, 7, 64, 3, 3, (2, 2), (1, 1)),
    (1, 3, 12, 10, 3, 3, (2, 2), (1, 1)),
    (1, 2, 6, 72, 3, 3, (2, 2), (1, 1)),
    # wider than 64 columns: column segments, the segment ends fetch their neighbour's dword
    (1, 3, 10, 112, 3, 3, (1, 1), (1, 1)),
    (2, 2, 70, 128, 3, 3, (1, 1), (1, 1)),
    (1, 2, 5, 68, 3, 3, (1, 1), (1, 1)),
    (1, 3, 20, 112, 3, 3, (2, 2), (1, 1)),
    (2, 2, 7, 200, 3, 3, (2, 2), (1, 1)),
    (1, 2, 5, 132, 3, 3, (2, 2), (1, 1)),
    # small planes (W <= 16): several planes share a DPP row; rows start at any byte
    (2, 6, 14, 14, 3, 3, (1, 1), (1, 1)),
    (3, 5, 7, 7, 3, 3, (1, 1), (1, 1)),
    (1, 4, 16, 16, 3, 3, (1, 1), (1, 1)),
    (2, 3, 9, 10, 3, 3, (1, 1), (1, 1)),
    (1, 7, 5, 3, 3, 3, (1, 1), (1, 1)),
    (1, 2, 64, 13, 3, 3, (1, 1), (1, 1)),
    (1, 37, 4, 8, 3, 3, (1, 1), (1, 1)),
    (1, 3, 1, 1, 3, 3, (1, 1), (1, 1)),
    # channel counts that are multiples of 4: the channel-last kernel (its NCHW twins take other paths)
    (2, 8, 9, 11, 3, 3, (1, 1), (1, 1)),
    (1, 12, 20, 7, 3, 3, (1, 1), (1, 1)),
    (1, 144, 14, 14, 3, 3, (1, 1), (1, 1)),
    (2, 4, 5, 37, 3, 3, (1, 1), (1, 1)),
    (1, 32, 3, 8, 3, 3, (1, 1), (1, 1)),
]


@pytest.mark.parametrize("case", DW_CASES)
@pytest.mark.parametrize("adt,za", [(np.uint8, 128), (np.uint8, 9), (np.int8, 0), (np.int8, 11)])
def test_depthwise(case, adt, za):
    B, C, H, W, KH, KW, stride, pad = case
    rng = np.random.default_rng(abs(hash((case, za))) % 2 ** 31)
    a = rnd_act(rng, (B, C, H, W), adt)
    w = rnd_w(rng, (C, 1, KH, KW))
    bias = rng.integers(-5000, 5000, C).astype(np.int32)
    mult, shift = datagen.requant_params(rng, np.full(C, 74.0 * 73.0 * np.sqrt(KH * KW)), 40.0)
    a_t, w_t = act_qtype(a, za), hago.QType(hago.I8)
    for acc_dt_r, acc_dt_g in ((ref.I32, hago.I32), (ref.I16, hago.I16)):
        want = ref.qconv2d(a, za, w, bias, ref.NCHW, stride, pad, C, acc_dt_r)
        got = qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), hago.NCHW, stride, pad, C, acc_dt_g)
        assert_same(host(got), want, f"depthwise raw {case}")
    want = ref.qconv2d(a, za, w, bias, ref.NCHW, stride, pad, C, ref.I32, ref_requant(mult, shift))
    got = qconv2d(dev(a), a_t, dev(w), w_t, dev(bias), hago.NCHW, stride, pad, C, hago.I32, gpu_requant(mult, shift))
    assert_same(host(got), want, f"depthwise rq {case}")
    want = ref.qconv2d(a.transpose(0, 2, 3, 1), za, w.transpose(0, 2, 3, 1), bias, ref.NHWC, stride, pad, C, ref.I32,
                       ref_requant(mult, shift))
    got = qconv2d(dev(a.transpose(0, 2, 3, 1)), a_t, dev(w.transpose(0, 2, 3, 1)), w_t, dev(bias), hago.NHWC,
                       stride, pad, C, hago.I32, gpu_requant(mult, shift))
    assert_same(host(got), want, f"depthwise nhwc {case}")
    # channel-last: raw int32, raw int16 and int16 accumulation with requantize
    an, wn = np.ascontiguousarray(a.transpose(0, 2, 3, 1)), np.ascontiguousarray(w.transpose(0, 2, 3, 1))
    for acc_dt_r, acc_dt_g in ((ref.I32, hago.I32), (ref.I16, hago.I16)):
        want = ref.qconv2d(an, za, wn, bias, ref.NHWC, stride, pad, C, acc_dt_r)
        got = qconv2d(dev(an), a_t, dev(wn), w_t, dev(bias), hago.NHWC, stride, pad, C, acc_dt_g)
        assert_same(host(got), want, f"depthwise nhwc raw {case}")
    m16, s16 = datagen.requant_params(rng, np.full(C, 19000.0), 40.0)
    want = ref.qconv2d(an, za, wn, bias, ref.NHWC, stride, pad, C, ref.I16, ref_requant(m16, s16))
    got = qconv2d(dev(an), a_t, dev(wn), w_t, dev(bias), hago.NHWC, stride, pad, C, hago.I16, gpu_requant(m16, s16))
    assert_same(host(got), want, f"depthwise nhwc int16 accumulation, requantized {case}")


@pytest.mark.parametrize("out_u8,z_out", [(False, 0), (False, -7), (True, 131)])
@pytest.mark.parametrize("with_bias", [True, False])
def test_depthwise_requant_constant_ranges(out_u8, z_out, with_bias):
    """The register kernel folds a channel's bias term, rounding term and output zero point into one 64-bit
    constant when they are small enough and takes its general form otherwise; both kinds of channel, and the
    bounds between them, in one launch."""
    B, C, H, W = 2, 12, 23, 24
    rng = np.random.default_rng(77 + z_out)
    a = rnd_act(rng, (B, C, H, W), np.uint8)
    w = rnd_w(rng, (C, 1, 3, 3))
    bias = rng.integers(-5000, 5000, C).astype(np.int64)
    bias[4], bias[5], bias[6], bias[7] = 2 ** 30 + 12345, -(2 ** 30) - 999, 2 ** 31 - 1, -(2 ** 31)
    bias[10], bias[11] = 2 ** 30 - 200000, -(2 ** 30) + 200000
    bias = bias.astype(np.int32)
    shift = np.array([0, 1, 5, 19, 20, 31, 3, 3, 19, 20, 30, 30], np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, size=C).astype(np.int32)
    a_t, w_t = act_qtype(a, 128), hago.QType(hago.I8)
    b_ref, b_gpu = (bias, dev(bias)) if with_bias else (None, None)
    want = ref.qconv2d(a, 128, w, b_ref, ref.NCHW, (1, 1), (1, 1), C, ref.I32, ref_requant(mult, shift, out_u8, z_out))
    got = qconv2d(dev(a), a_t, dev(w), w_t, b_gpu, hago.NCHW, (1, 1), (1, 1), C, hago.I32,
                       gpu_requant(mult, shift, out_u8, z_out))
    assert_same(host(got), want, "depthwise per-channel")
    assert len(np.unique(want)) > 50
    # one multiplier and shift for the whole tensor
    want = ref.qconv2d(a, 128, w, b_ref, ref.NCHW, (1, 1), (1, 1), C, ref.I32,
                       ref_requant(mult[:1], np.array([9], np.int32), out_u8, z_out))
    got = qconv2d(dev(a), a_t, dev(w), w_t, b_gpu, hago.NCHW, (1, 1), (1, 1), C, hago.I32,
                       gpu_requant(mult[:1], np.array([9], np.int32), out_u8, z_out))
    assert_same(host(got), want, "depthwise per-tensor")


def test_empty_inputs_are_a_no_op():
    a = torch.empty((0, 16), dtype=torch.uint8, device=DEV)
    w = torch.zeros((8, 16), dtype=torch.int8, device=DEV)
    out = hago.qdense(a, hago.QType(hago.U8, zero_point=128), w, hago.QType(hago.I8))
    assert out.shape == (0, 8)
    x = torch.empty((0, 3, 4), dtype=torch.float32, device=DEV)
    y = hago.simquant(x, torch.ones(3, device=DEV), torch.zeros(3, dtype=torch.int32, device=DEV), hago.QType(hago.I8))
    assert y.numel() == 0
    a4 = torch.empty((0, 4, 5, 5), dtype=torch.int8, device=DEV)
    w4 = torch.zeros((4, 4, 3, 3), dtype=torch.int8, device=DEV)
    out = qconv2d(a4, hago.QType(hago.I8), w4, hago.QType(hago.I8), pad=(1, 1))
    assert out.shape == (0, 4, 5, 5)
    torch.cuda.synchronize()


def test_results_are_deterministic():
    c = datagen.config5_layer(1, M=512)
    args = (dev(c["a"]), act_qtype(c["a"], c["z_a"]), dev(c["w"]), hago.QType(hago.I8), dev(c["bias"]), hago.I32)
    rq = gpu_requant(c["mult"], c["shift"])
    r1 = host(hago.qdense(*args, rq))
    r2 = host(hago.qdense(*args, rq))
    assert np.array_equal(r1, r2)
