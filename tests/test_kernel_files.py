"""A process loads all kernels of a file when it calls the first of them, so kernels for different kinds of results lie in files of their own; and none of
the kernels whose loops are written to the last register spills any."""
import glob
import os
import re

import pytest

from paper_2103_14949_amd import build


# (the kind of results is the last template argument of the first three; the streaming kernels of one tile have one name in every file)
@pytest.mark.parametrize("kernel, most", [("conv3x3_nchw_kernel", 72), ("conv_direct_kernel", 26), ("qgemm_line_kernel", 6), ("qgemm_dma_kernel", 42)])
def test_one_kind_of_results_per_file(kernel, most):
    paths = glob.glob(os.path.join(os.path.dirname(build.LIB), "_build", "*gfx950.s"))
    if not paths:
        pytest.skip("no assembly here: the libraries were built elsewhere")
    sources = {os.path.basename(s)[:-len(".hip")] for s in build.sources()}
    files = 0
    for path in paths:
        if os.path.basename(path).split("-hip-")[0] not in sources:
            continue
        with open(path) as f:
            text = f.read()
        names = re.findall(r"^\s*\.amdhsa_kernel (\S*" + kernel + r"I\S*)", text, re.M)
        files += bool(names)
        assert len(names) <= most, (path, len(names))
        if kernel != "qgemm_dma_kernel":
            assert len({re.search(r"Li(\d+)EEE?v", n)[1] for n in names}) <= 1, path
        if kernel not in ("conv_direct_kernel", "qgemm_line_kernel"):
            continue
        spilled = re.findall(r"\.name:\s+(\S*" + kernel + r"I\S*).*?\.vgpr_spill_count:\s+(\d+)", text, re.S)
        assert len(spilled) == len(names) and [n for n, count in spilled if int(count)] == []
    assert files >= 3
