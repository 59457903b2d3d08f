"""Dense layers on the large tiles whose operands stream in stages of 128 bytes: reductions that end inside a stage, at its
end and right behind it, one stage and many, ragged rows and channels, and every kind of result."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [0, 1, 5, 6])  # 256 x 256, 192 x 256, 128 x 256; 64 x 64
@pytest.mark.parametrize("K", [16, 48, 112, 128, 144, 240, 256, 272, 384, 400, 1040])
def test_stage_edges(tile, K):
    rng = np.random.default_rng(100 * K + tile)
    hago.set_test_hook(hago.HOOK_STREAM_TILE, tile)
    try:
        for M, N, act_u8 in ((300, 208, True), (257, 401, False), (1, 16, True), (512, 37, True), (70, 399, True)):
            a = rng.integers(0, 256, (M, K)).astype(np.uint8) if act_u8 else rng.integers(-128, 128, (M, K)).astype(np.int8)
            za = 131 if act_u8 else -7
            w = rng.integers(-127, 128, (N, K)).astype(np.int8)
            bias = rng.integers(-3000, 3000, N).astype(np.int32)
            mult = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32)
            shift = rng.integers(8, 12, N).astype(np.int32)
            args = dev(a), act_qtype(a, za), dev(w), hago.QType(hago.I8), dev(bias)
            for acc, racc in ((hago.I32, ref.I32), (hago.I16, ref.I16)):
                assert_same(host(hago.qdense(*args, acc)), ref.qdense(a, za, w, bias, racc), f"raw {M, N, K, acc}")
            # one channel in its first 32 with a shift that the folded (0) or the saturating form (22) does not take
            for special in (None, 0, 22):
                sh = shift.copy()
                if special is not None:
                    sh[min(21, N - 1)] = special
                for out_u8, z, clip in ((False, 5, (-128, 127)), (False, 5, (-100, 90)), (True, 131, (0, 255))):
                    assert_same(host(hago.qdense(*args, hago.I32, gpu_requant(mult, sh, out_u8, z, clip))),
                                ref.qdense(a, za, w, bias, ref.I32, ref_requant(mult, sh, out_u8, z, clip)), f"{M, N, K, out_u8, clip, special}")
    finally:
        hago.set_test_hook(hago.HOOK_STREAM_TILE, -1)
