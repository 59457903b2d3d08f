"""Aligned dense layers of every kernel that serves them, on both sides of the lines between them (tests/test_dense_routes.py has
which is which): the few-tile kernel with four and eight wavefronts, and 64 x 64 tiles with stages of 64 and 128 bytes, whole and
with a reduction that ends inside one, over one round of the chip and more; requantized and raw."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu


# one kernel for all of them: few tiles
FEW = [
    (4, 64, 48), (5, 64, 48), (4, 320, 48), (3, 16, 16), (33, 112, 37),
    (16, 640, 40), (17, 640, 40), (16, 512, 40), (40, 768, 33), (40, 1024, 33), (40, 1152, 33), (16, 1152, 33),
    (8192, 80, 32), (8193, 80, 32),                             # one round of tiles over the chip, and one more tile
    (160, 7168, 832), (128, 7168, 1024), (40, 7040, 64),        # very long
    (1000, 2880, 512), (360, 2080, 720), (2048, 1472, 130),
]
# 527 tiles of 32 x 32 and more, where the line to the few-tile kernel is one of the reduction's length: (that kernel, the other)
OF_LENGTH = [((544, 80, 992), (544, 64, 992)), ((544, 640, 992), (544, 656, 992))]
# 64 x 64 tiles with 64-byte and with 128-byte stages
STAGES_64 = [(544, 64, 992), (544, 656, 992), (544, 704, 992), (544, 752, 992), (544, 832, 992), (544, 2032, 992), (700, 1344, 1216)]
STAGES_128 = [(544, 768, 992), (544, 896, 992), (544, 2064, 992), (1024, 768, 2048)]
LARGER = [(1088, 768, 2048), (1565, 384, 2496)]                 # more than two rounds of 64 x 64


@pytest.mark.parametrize("M,K,N", FEW + [x for x, _ in OF_LENGTH] + STAGES_64 + STAGES_128 + LARGER)
def test_both_sides(M, K, N):
    rng = np.random.default_rng(M + 3 * K + 7 * N)
    a, w = rng.integers(0, 256, (M, K)).astype(np.uint8), rng.integers(-127, 128, (N, K)).astype(np.int8)
    bias = rng.integers(-10 ** 5, 10 ** 5, N).astype(np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32)
    shift = rng.integers(9, 13, N).astype(np.int32)
    args = dev(a), act_qtype(a, 121), dev(w), hago.QType(hago.I8), dev(bias)
    sums = ref.qdense(a, 121, w, bias)
    assert_same(host(hago.qdense(*args)), sums, "raw")
    assert_same(host(hago.qdense(*args, hago.I16)), sums.astype(np.int16), "raw 16")
    for out_u8, z, clip in ((False, -3, (-128, 127)), (True, 131, (0, 255)), (False, 0, (-100, 90))):
        want = ref.requantize(np.ascontiguousarray(sums.reshape(M, N, 1)), ref_requant(mult, shift, out_u8, z, clip)).reshape(M, N)
        assert_same(host(hago.qdense(*args, hago.I32, gpu_requant(mult, shift, out_u8, z, clip))), want, f"{out_u8, z, clip}")
