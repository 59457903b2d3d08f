"""Sums that go out as 32 or 16 bits, by quads and sixteens of lanes: rows and images that begin with a line, at 16 bytes, at 4
and anywhere, tiles that end inside a piece, in every kernel that writes them so."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403

ACCS = [(hago.I32, ref.I32, torch.int32), (hago.I16, ref.I16, torch.int16)]


# (few tiles; unaligned rows in 64 and 128 tiles; 64 x 64 tiles; 256-wide ones)
@pytest.mark.parametrize("m, k", [(70, 64), (45, 131), (1500, 701), (4500, 129), (1100, 768), (4000, 512)])
@pytest.mark.parametrize("n", [40, 101, 130, 208, 516])
def test_dense(m, k, n):
    rng = np.random.default_rng(m + k + n)
    a, w = rng.integers(0, 256, (m, k)).astype(np.uint8), rng.integers(-127, 128, (n, k)).astype(np.int8)
    bias = rng.integers(-5000, 5000, n).astype(np.int32)
    args = dev(a), act_qtype(a, 131), dev(w), hago.QType(hago.I8), dev(bias)
    for acc, racc, dtype in ACCS:
        want = ref.qdense(a, 131, w, bias, racc)
        for off in (0, 4, 1):
            got = into_guard(lambda out: hago.qdense(*args, acc, out=out), (m, n), torch.from_numpy(want[:1]).dtype, off)
            assert_same(got, want, f"{m, n, k, dtype} off {off}")


@pytest.mark.parametrize("tile", [0, 1, 3, 5, 6])
def test_dense_tiles(tile):
    rng = np.random.default_rng(tile)
    hago.set_test_hook(hago.HOOK_STREAM_TILE, tile)
    try:
        for m, n, k in ((300, 208, 64), (257, 404, 128), (512, 37, 192), (70, 402, 256)):
            a, w = rng.integers(0, 256, (m, k)).astype(np.uint8), rng.integers(-127, 128, (n, k)).astype(np.int8)
            args = dev(a), act_qtype(a, 9), dev(w), hago.QType(hago.I8), None
            for acc, racc, dtype in ACCS:
                assert_same(host(hago.qdense(*args, acc)), ref.qdense(a, 9, w, None, racc), f"{m, n, k, dtype}")
    finally:
        hago.set_test_hook(hago.HOOK_STREAM_TILE, -1)


# images and output channels of whole pieces, of half ones and of none; several column segments; tiles that span images
@pytest.mark.parametrize("geometry", [(3, 3, 64, 60, 64, 5, 1), (2, 3, 33, 31, 72, 7, 2), (5, 64, 17, 24, 70, 3, 2), (9, 48, 14, 14, 96, 3, 2),
                                      (2, 5, 20, 150, 40, 5, 1), (4, 160, 28, 28, 136, 3, 1), (6, 128, 20, 20, 128, 3, 1), (7, 96, 9, 13, 100, 5, 1)])
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_convolution(geometry, layout):
    B, C, H, W, O, k, s = geometry
    rng = np.random.default_rng(1000 * W + O)
    ashape, wshape = ((B, C, H, W), (O, C, k, k)) if layout == "nchw" else ((B, H, W, C), (O, k, k, C))
    a, w = rng.integers(0, 256, ashape).astype(np.uint8), rng.integers(-127, 128, wshape).astype(np.int8)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, O).astype(np.int32), rng.integers(7, 12, O).astype(np.int32)
    geo, rgeo = (((hago.NCHW if layout == "nchw" else hago.NHWC), (s, s), (k // 2, k // 2), 1),
                 ((ref.NCHW if layout == "nchw" else ref.NHWC), (s, s), (k // 2, k // 2), 1))
    args = (dev(a), act_qtype(a, 131), dev(w), hago.QType(hago.I8), None, *geo)
    need = hago.qconv2d_workspace_bytes(a.shape, w.shape, *geo)
    for acc, racc, dtype in ACCS:
        for rq, rrq in ((None, None), (gpu_requant(mult, shift), ref_requant(mult, shift))):
            want = ref.qconv2d(a, 131, w, None, *rgeo, racc, rrq)
            for off in (0, 4, 1):
                for ws in (None, torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)):
                    got = into_guard(lambda out: hago.qconv2d(*args, acc, rq, workspace=ws, out=out), want.shape,
                                     torch.from_numpy(want[:1]).dtype, off)
                    assert_same(got, want, f"{geometry} {layout} {dtype} {rq is None} off {off}")
