"""The dense kernel of few tiles: reductions that end at, in front of and behind a block of 128 bytes of a row, with fewer and
more blocks than wavefronts and than a ring of two for each, rows at every offset from four bytes in a buffer of other values,
zero points at both ends of their range, rows and channels that end inside a tile."""
import numpy as np
import pytest

from gpu_util import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu


def inside(x, offset):
    """The tensor on the GPU, `offset` elements into a buffer that holds other values on both sides of it."""
    flat = torch.full((x.size + offset + 300,), 113, dtype=torch.from_numpy(x).dtype, device=DEV)
    view = flat[offset: offset + x.size].view(x.shape)
    view.copy_(dev(x))
    return view


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("KB", [1, 15, 16, 31, 33, 64, 96, 127, 128, 129, 250, 256, 500, 512, 513, 640, 1023, 1024, 1025, 1150,
                                2047, 2048, 2050, 2177, 3200])
def test_ends_of_blocks(KB, form, gemm_path):
    rng = np.random.default_rng(KB)
    i8, i16 = hago.QType(hago.I8), hago.QType(hago.I16, 16, True, -7)
    gemm_path(1)
    hago.set_test_hook(hago.HOOK_GENERAL_TILE, form)
    try:
        for M, N, oa, ow in ((32, 32, 0, 0), (33, 5, 4, 8), (1, 67, 1, 3), (70, 31, 2, 0)):
            mult, shift = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32), rng.integers(5, 15, N).astype(np.int32)
            bias = rng.integers(-3000, 3000, N).astype(np.int32)
            a, w = rng.integers(0, 256, (M, KB)).astype(np.uint8), rng.integers(-128, 128, (N, KB)).astype(np.int8)
            for z in (0, 128, 255):
                got = hago.qdense(inside(a, oa), hago.QType(hago.U8, 8, False, z), inside(w, ow), i8, dev(bias), hago.I32,
                                  gpu_requant(mult, shift))
                assert_same(host(got), ref.qdense(a, z, w, bias, ref.I32, ref_requant(mult, shift)), f"uint8 {M, N, oa, ow} {z}")
            if KB % 2 == 0:
                a, w = (rng.integers(-32768, 32768, s).astype(np.int16) for s in ((M, KB // 2), (N, KB // 2)))
                got = hago.qdense(inside(a, oa), i16, inside(w, ow), hago.QType(hago.I16, 16, True, 0), dev(bias), hago.I32)
                assert_same(host(got), ref.qdense(a, -7, w, bias, ref.I32, None), f"int16 {M, N, oa, ow}")
    finally:
        hago.set_test_hook(hago.HOOK_GENERAL_TILE, -1)


@pytest.mark.parametrize("M,K,N", [(512, 65, 1024), (513, 640, 1024), (1000, 64, 1000), (257, 512, 7168), (1025, 1280, 1000), (30, 100, 57350)])
def test_lines_to_the_larger_tiles(M, K, N):
    """On both sides of the numbers of tiles at which another kernel takes over; the results of some rows and channels."""
    rng = np.random.default_rng(M + K)
    a, w = rng.integers(-128, 128, (M, K)).astype(np.int8), rng.integers(-128, 128, (N, K)).astype(np.int8)
    for cut_m, cut_n in ((0, 0), (1, 0), (0, 8), (M // 2, 0)):
        got = host(hago.qdense(dev(a[cut_m:]), hago.QType(hago.I8, 8, True, 3), dev(w[cut_n:]), hago.QType(hago.I8)))
        rows, cols = rng.integers(0, M - cut_m, 40), rng.integers(0, N - cut_n, 40)
        rows[0], cols[0] = M - cut_m - 1, N - cut_n - 1
        assert_same(got[np.ix_(rows, cols)], ref.qdense(a[cut_m:][rows], 3, w[cut_n:][cols], None, ref.I32, None), f"{cut_m, cut_n}")
