"""Results too large for the ways of small ones: depthwise layers of several column segments and of ragged rows, 32-bit sums of the one-launch 3x3
kernel, dense rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403


@pytest.mark.parametrize("case", [(10, 90, 112, 112), (10, 90, 113, 111), (48, 140, 41, 41), (30, 130, 50, 56)])
@pytest.mark.parametrize("act_u8", [False, True])
def test_depthwise(case, act_u8):
    B, C, H, W = case
    rng = np.random.default_rng(W + act_u8)
    a = rng.integers(0, 256, case).astype(np.uint8) if act_u8 else rng.integers(-127, 128, case).astype(np.int8)
    w, za = rng.integers(-127, 128, (C, 1, 3, 3)).astype(np.int8), 131 if act_u8 else 0
    mult, shift = rng.integers(2 ** 30, 2 ** 31, C).astype(np.int32), rng.integers(7, 12, C).astype(np.int32)
    want = ref.qconv2d(a, za, w, None, ref.NCHW, (1, 1), (1, 1), C, ref.I32, ref_requant(mult, shift))
    args = (dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), None, hago.NCHW, (1, 1), (1, 1), C, hago.I32, gpu_requant(mult, shift))
    for off in (0, 4, 1):
        assert_same(into_guard(lambda out: hago.qconv2d(*args, out=out), a.shape, torch.int8, off), want, f"{case} off {off}")


@pytest.mark.parametrize("B, O", [(50, 52), (40, 63)])   # 8.15 and 7.9 million sums, on both sides of the rule
def test_sums_3x3(B, O):
    rng = np.random.default_rng(B)
    a, w = rng.integers(-127, 128, (B, 32, 56, 56)).astype(np.int8), rng.integers(-127, 128, (O, 32, 3, 3)).astype(np.int8)
    want = ref.qconv2d(a, 0, w, None, ref.NCHW, (1, 1), (1, 1), 1, ref.I32)
    args = (dev(a), act_qtype(a, 0), dev(w), hago.QType(hago.I8), None, hago.NCHW, (1, 1), (1, 1), 1, hago.I32)
    for off in (0, 3):
        assert_same(into_guard(lambda out: hago.qconv2d(*args, out=out), want.shape, torch.int32, off), want, f"{B, O, off}")


@pytest.mark.parametrize("n", [960, 1024, 1001, 1040, 4100])   # 3.9 million results in whole lines, more, and rows of no whole lines
@pytest.mark.parametrize("m, k", [(4100, 128), (4100, 144)])
def test_dense(m, k, n):
    rng = np.random.default_rng(n + k)
    a, w = rng.integers(0, 256, (m, k)).astype(np.uint8), rng.integers(-127, 128, (n, k)).astype(np.int8)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, n).astype(np.int32), rng.integers(6, 10, n).astype(np.int32)
    args = (dev(a), act_qtype(a, 128), dev(w), hago.QType(hago.I8), None, hago.I32)
    for clip in ((-128, 127), (-100, 90)):
        want = ref.qdense(a, 128, w, None, ref.I32, ref_requant(mult, shift, clip=clip))
        for off in (0, 16, 1):
            assert_same(into_guard(lambda out: hago.qdense(*args, gpu_requant(mult, shift, clip=clip), out=out), (m, n), torch.int8, off),
                        want, f"{m}x{k}->{n} {clip} off {off}")
