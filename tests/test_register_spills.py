"""Kernels whose loops are written to the last register: none of theirs lies in scratch memory, as built."""
import glob
import os
import re

import pytest

from paper_2103_14949_amd import build


@pytest.mark.parametrize("source", ["conv_direct", "qgemm_line", "qgemm_any"])
def test_no_vector_register_is_spilled(source):
    paths = glob.glob(os.path.join(os.path.dirname(build.LIB), "_build", f"{source}-*gfx950.s"))
    if not paths:
        pytest.skip("no assembly here: the libraries were built elsewhere")
    with open(paths[0]) as f:
        text = f.read()
    kernels = re.findall(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", text, re.S)
    assert kernels and [k for k, spilled in kernels if int(spilled)] == []
