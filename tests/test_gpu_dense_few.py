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


# Layers on both sides of each line between this kernel and the larger tiles (tests/test_dense_routes.py): type, rows, reduction,
# channels, bytes into a buffer
FEW = [
    ("i8", 512, 768, 1024, 0), ("i8", 544, 80, 992, 0), ("i8", 544, 640, 992, 0), ("i8", 1024, 640, 1024, 0),       # whole chunks
    ("i8", 544, 640, 992, 4), ("u8", 1024, 511, 2048, 0), ("i8", 1056, 511, 1024, 0), ("u8", 1024, 767, 1024, 0), ("i8", 1024, 768, 1024, 1),
    ("u8", 7200, 926, 66, 0), ("i8", 20, 1001, 16500, 0), ("u8", 65536, 100, 20, 0),                                  # narrow
    ("i16", 512, 300, 1024, 0),
]
OTHERS = [
    ("i8", 544, 768, 992, 0), ("i8", 544, 64, 992, 0), ("i8", 544, 656, 992, 0), ("i8", 1025, 640, 1024, 0),
    ("i8", 1056, 640, 1024, 4), ("u8", 1025, 511, 2048, 0), ("i8", 1056, 513, 1024, 0), ("u8", 1024, 769, 1024, 0), ("i8", 1056, 528, 1024, 1),
    ("u8", 7200, 926, 98, 0), ("u8", 7200, 1025, 66, 0), ("u8", 65537, 100, 20, 0),
    ("i16", 544, 300, 992, 0),
]


@pytest.mark.parametrize("act,M,K,N,offset", FEW + OTHERS)
def test_lines_to_the_larger_tiles(act, M, K, N, offset):
    """The results of some rows and channels, the last ones among them."""
    rng = np.random.default_rng(M + K)
    dtype, top = {"u8": (np.uint8, 256), "i8": (np.int8, 128), "i16": (np.int16, 32768)}[act]
    a = rng.integers(0 if act == "u8" else -top, top, (M, K)).astype(dtype)
    w = rng.integers(-32768 if act == "i16" else -128, 32768 if act == "i16" else 128, (N, K)).astype(np.int16 if act == "i16" else np.int8)
    a_t, w_t = (hago.QType(hago.I16, 16, True, 3), hago.QType(hago.I16, 16, True, 0)) if act == "i16" else (act_qtype(a, 3), hago.QType(hago.I8))
    mult, shift = rng.integers(2 ** 30, 2 ** 31, N, dtype=np.int64).astype(np.int32), rng.integers(8, 15, N).astype(np.int32)
    rows, cols = rng.integers(0, M, 40), rng.integers(0, N, 40)
    rows[:2], cols[:2] = (M - 1, M - 2), (N - 1, N - 2)
    rr = ref_requant(mult[cols], shift[cols])
    da, dw = inside(a, offset), dev(w)
    assert_same(host(hago.qdense(da, a_t, dw, w_t))[np.ix_(rows, cols)], ref.qdense(a[rows], 3, w[cols], None, ref.I32, None), "raw")
    got = host(hago.qdense(da, a_t, dw, w_t, None, hago.I32, gpu_requant(mult, shift)))
    assert_same(got[np.ix_(rows, cols)], ref.qdense(a[rows], 3, w[cols], None, ref.I32, rr), "requantized")
