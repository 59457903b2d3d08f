"""Dense layers whose rows start off multiples of four bytes (loaded from the aligned dwords that hold them), at every
offset of the tensors, in every form of that kernel, with the saturating requantize of its staged form: shifts on both sides
of what it takes, sums that wrap, whole and narrower clips."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu


def at_offset(x, elements):
    """The tensor on the GPU, `elements` behind the start of an allocation."""
    flat = torch.zeros(x.size + elements + 16, dtype=torch.from_numpy(x).dtype, device=DEV)
    view = flat[elements: elements + x.size].view(x.shape)
    view.copy_(dev(x))
    return view


@pytest.mark.parametrize("form", [-1, 0, 1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K", [(33, 35, 97), (70, 67, 131), (3, 130, 257), (65, 40, 320)])
def test_offsets(M, N, K, form, gemm_path):
    rng = np.random.default_rng(M + 7 * N + 31 * K)
    bias = rng.integers(-3000, 3000, N).astype(np.int32)
    mult = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32)
    a8, w8 = rng.integers(0, 256, (M, K)).astype(np.uint8), rng.integers(-127, 128, (N, K)).astype(np.int8)
    a16 = rng.integers(-32768, 32768, (M, K)).astype(np.int16)
    w16 = rng.integers(-32768, 32768, (N, K)).astype(np.int16)
    w_t, i16 = hago.QType(hago.I8), lambda z: hago.QType(hago.I16, 16, True, z)
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, form)
    try:
        for oa, ow in ((0, 0), (1, 2), (2, 3), (3, 0)):
            for out_u8, z, clip, s8, s16 in ((False, -9, (-128, 127), (6, 10), (18, 21)), (True, 200, (0, 255), (1, 22), (20, 22)),
                                             (False, 3, (-100, 127), (6, 10), (18, 21))):
                for a, w, za, sh, types in ((a8, w8, 119, s8, (hago.QType(hago.U8, zero_point=119), w_t)),
                                            (a16, w16, -250, s16, (i16(-250), i16(0)))):
                    shift = rng.integers(sh[0], sh[1] + 1, N).astype(np.int32)
                    got = hago.qdense(at_offset(a, oa), types[0], at_offset(w, ow), types[1], dev(bias), hago.I32,
                                      gpu_requant(mult, shift, out_u8, z, clip))
                    assert_same(host(got), ref.qdense(a, za, w, bias, ref.I32, ref_requant(mult, shift, out_u8, z, clip)),
                                f"{a.dtype} offsets {oa, ow} {out_u8, z, clip, sh}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)
