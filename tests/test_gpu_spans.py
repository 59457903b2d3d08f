"""Channel-last and ragged tensors at the edges of their division into spans: max-abs with few, some and many spans of a workgroup, and candidates
on both sides of the number from which whole lines are worth longer rounds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403


# (spans of a workgroup: 1, 4, 8, 16, 24 and, from 32 on not rounded to fours, 36 and 57)
@pytest.mark.parametrize("shape", [(3000, 37, 1), (8000, 64, 1), (20000, 51, 1), (65536, 45, 1), (500000, 3, 1), (60000, 30, 4), (200000, 37, 1),
                                   (300000, 64, 1), (710001, 37, 1)])
def test_absmax(shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(shape[0] + shape[1])
    x = torch.randn(shape, generator=g, device=DEV)
    for c in range(shape[1]):   # each channel's largest where a span, a workgroup or the tensor may end
        o = (shape[0] - 1 - c, c, (shape[0] // 2 + 7 * c) % shape[0])[c % 3]
        x[o, c, c % shape[2]] = (-1) ** c * (8.0 + c)
    assert_same_bits(host(hago.absmax(x)), 8.0 + np.arange(shape[1], dtype=np.float32), f"{shape}")


@pytest.mark.parametrize("shape", [(20000, 10, 9), (17000, 3, 9), (70000, 3, 1), (9000, 7, 7), (24000, 45, 1)])
@pytest.mark.parametrize("n", [5, 6, 8])
def test_candidates(shape, n):
    rng = np.random.default_rng(shape[0] + n)
    x = (rng.standard_normal(shape) * 2).astype(np.float32)
    scales = rng.uniform(0.01, 0.05, (n, shape[1])).astype(np.float32)
    zps = rng.integers(-9, 10, (n, shape[1])).astype(np.int32)
    lo, hi = [-(1 << (7 - b % 4)) for b in range(n)], [(1 << (7 - b % 4)) - 1 for b in range(n)]
    guard = torch.full((n * x.size + 64,), 77.0, device=DEV)
    hago.simquant_batched(dev(x), dev(scales), dev(zps), hago.QType(hago.I8), lo, hi, out=guard[:n * x.size].view(n, *shape))
    assert int((guard[n * x.size:] != 77).sum()) == 0
    got = host(guard[:n * x.size].view(n, *shape))
    for b in range(n):
        assert_same_bits(got[b], ref.simquant(x, scales[b], zps[b], lo[b], hi[b]), f"{shape} candidate {b} of {n}")
