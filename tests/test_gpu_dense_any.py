"""GPU parity of the dense layer on operands of any size and alignment (rows that start at any byte, reductions that
end inside a chunk) and on int16 operands, in every form of that kernel, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403
from paper_2103_14949_amd import datagen

# K: shorter than a chunk; one short of / one past a chunk, a 32-k group, a stage; several stages with every kind of tail
SIZES = [(1, 1, 15), (33, 31, 17), (65, 129, 31), (64, 64, 33), (129, 66, 127), (70, 130, 129), (200, 257, 255),
         (31, 95, 511), (130, 65, 643), (5, 300, 1283)]


@pytest.mark.parametrize("form", [-1, 0, 1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_every_form_and_tail(M, N, K, form, gemm_path):
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    bias = rng.integers(-10 ** 5, 10 ** 5, N).astype(np.int32)
    a, w = rng.integers(0, 256, (M, K)).astype(np.uint8), rng.integers(-128, 128, (N, K)).astype(np.int8)
    a16 = rng.integers(-32768, 32768, (M, K)).astype(np.int16)
    w16 = rng.integers(-32768, 32768, (N, K)).astype(np.int16)
    mult, shift = datagen.requant_params(rng, np.full(N, 74.0 * 73.0 * np.sqrt(K)), 40.0)
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, form)
    try:
        rr, rg = ref_requant(mult, shift, True, 10, (10, 255), 1), gpu_requant(mult, shift, True, 10, (10, 255), rounding=1)
        w_t, i16 = hago.QType(hago.I8), lambda z: hago.QType(hago.I16, 16, True, z)
        assert_same(host(hago.qdense(dev(a), act_qtype(a, 131), dev(w), w_t, dev(bias), hago.I32, rg)),
                    ref.qdense(a, 131, w, bias, ref.I32, rr), "requantized")
        assert_same(host(hago.qdense(dev(a), act_qtype(a, 3), dev(w), w_t, dev(bias))), ref.qdense(a, 3, w, bias), "raw")
        assert_same(host(hago.qdense(dev(a), act_qtype(a, 3), dev(w), w_t, None, hago.I16)), ref.qdense(a, 3, w, None, ref.I16), "raw 16")
        for z in (0, -300):
            assert_same(host(hago.qdense(dev(a16), i16(z), dev(w16), i16(0), dev(bias))), ref.qdense(a16, z, w16, bias), f"int16 z={z}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)
