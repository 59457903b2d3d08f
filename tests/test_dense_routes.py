"""Which kernel serves a dense layer, on the CPU: the sizes that the GPU tests of a kernel, and of the lines between two, run at are
those that reach it."""
import pytest

import test_gpu_dense_few as few
import test_gpu_dense_lines as lines


def dense(act, M, K, N, offset=0, raw=0):
    return f"dense {act} {M} {K} {N} {raw} {offset}"


def served(routes, calls):
    found = routes(calls)
    assert all(len(k) == 1 for k in found), found
    return [k[0] for k in found]


@pytest.mark.parametrize("raw", [0, 1])
def test_layers_of_whole_chunks(routes, raw):
    at = lambda sizes: served(routes, [dense("u8", *s, raw=raw) for s in sizes])  # noqa: E731
    assert {k[:k.index("<")] for k in at(lines.FEW + [x for x, _ in lines.OF_LENGTH])} == {"qgemm_few_kernel"}
    assert {k.split(",")[2] for k in at(lines.FEW)} == {"4>", "8>"}      # wavefronts
    tiles_64 = "qgemm_dma_kernel<2,2,1,1,4,2,0,false,true,"
    assert set(at(lines.STAGES_64)) == {tiles_64 + "true,64>", tiles_64 + "false,64>"}      # (reductions of whole stages, and others)
    assert set(at(lines.STAGES_128)) == {tiles_64 + "true,128>", tiles_64 + "false,128>"}
    assert not any(k.startswith((tiles_64, "qgemm_few")) for k in at(lines.LARGER[:1]))
    for here, there in lines.OF_LENGTH:
        assert at([here]) != at([there])


def test_lines_to_the_larger_tiles(routes):
    calls = [dense(*x) for x in few.FEW + few.OTHERS]
    for call, kernel in zip(calls, served(routes, calls)):
        assert kernel.startswith("qgemm_few") == (call in calls[:len(few.FEW)]), (call, kernel)


def test_narrow_accumulators_of_any_size(routes):
    """Whole-range codes of a 16- or 24-bit accumulator: a kernel of their own on the large tiles."""
    kernels = {(size, bits): served(routes, [f"dense i8 {size} 0 0 {bits}"])[0] for size in ("3000 101 1984", "2000 700 1003") for bits in (32, 24, 16)}
    large, small = ("qgemm_staged_kernel<false,2,4,2,1,1,", "qgemm_staged_kernel<false,2,2,1,1,2,")
    assert kernels["3000 101 1984", 16] == kernels["3000 101 1984", 24] != kernels["3000 101 1984", 32]
    assert all(kernels["3000 101 1984", b].startswith(large) and kernels["2000 700 1003", b].startswith(small) for b in (32, 24, 16))
    assert kernels["3000 101 1984", 16][len(large):] not in {kernels["2000 700 1003", b][len(small):] for b in (32, 24, 16)}
