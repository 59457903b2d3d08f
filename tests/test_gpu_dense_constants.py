"""The dense kernel that splits one 32 x 32 tile over wavefronts: channels that end inside a thread's four, bias and requantize
parameters that are there or not, one for all channels or one each."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("N", [1, 3, 31, 32, 33, 66])
def test_channel_constants(N, form, gemm_path):
    rng = np.random.default_rng(10 * N + form)
    M, K = 35, 70
    a8, w8 = rng.integers(-128, 128, (M, K)).astype(np.int8), rng.integers(-127, 128, (N, K)).astype(np.int8)
    a16, w16 = rng.integers(-900, 900, (M, K)).astype(np.int16), rng.integers(-900, 900, (N, K)).astype(np.int16)
    bias = rng.integers(-30000, 30000, N).astype(np.int32)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32), rng.integers(6, 20, N).astype(np.int32)
    i8, i16 = hago.QType(hago.I8), hago.QType(hago.I16, 16, True, 0)
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, form)
    try:
        for a, w, t in ((a8, w8, i8), (a16, w16, i16)):
            for b in (None, bias):
                for m, s in ((None, None), (mult, shift), (mult[:1], shift[:1]), (None, shift), (None, shift[:1])):
                    rg = None if s is None else hago.Requant(None if m is None else dev(m), dev(s), i8)
                    rr = None if s is None else ref.Requant(m, s)
                    assert_same(host(hago.qdense(dev(a), t, dev(w), t, dev(b), hago.I32, rg)), ref.qdense(a, 0, w, b, ref.I32, rr),
                                f"{a.dtype} bias {b is not None} {None if m is None else m.size} {None if s is None else s.size}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)
