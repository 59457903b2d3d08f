"""How many wavefronts of the 1x1 kernel's variants a SIMD has registers for, as the launch counts them and as built."""
import glob
import os
import re
import subprocess

import pytest

from paper_2103_14949_amd import build

REGISTERS = 512   # of a lane and SIMD, allocated in blocks of eight


def test_waves_per_simd(tmp_path):
    paths = glob.glob(os.path.join(os.path.dirname(build.LIB), "_build", "pointwise-*gfx950.s"))
    if not paths:
        pytest.skip("no assembly here: the libraries were built elsewhere")
    with open(os.path.join(build.CSRC, "pointwise.hip")) as f:
        rule = re.search(r"^constexpr int waves_per_simd\(.*?^}$", f.read(), re.S | re.M)[0]
    with open(paths[0]) as f:
        found = {tuple(map(int, m[:4])): int(m[4]) for m in re.findall(
            r"\.name:\s+\S*pw_nchw_kernelILi(\d)ELb(\d)ELi1ELi([23])ELb(\d)E\S*.*?\.vgpr_count:\s+(\d+)", f.read(), re.S)}
    assert len(found) == 4 * 2 * 2, found
    source = tmp_path / "rule.cpp"
    source.write_text("#include <cstdio>\n" + rule + "\nint main() {\n" + "".join(
        f'  std::printf("%d\\n", waves_per_simd({mode}, {acc16}, {ch}, {small}));\n' for mode, acc16, ch, small in found) + "}\n")
    subprocess.run(["g++", "-std=c++17", str(source), "-o", str(tmp_path / "rule")], check=True)
    counted = map(int, subprocess.run([str(tmp_path / "rule")], capture_output=True, text=True, check=True).stdout.split())
    assert dict(zip(found, counted)) == {k: REGISTERS // ((v + 7) // 8 * 8) for k, v in found.items()}


def test_waves_per_simd_of_every_kind_of_codes(tmp_path):
    paths = glob.glob(os.path.join(os.path.dirname(build.LIB), "_build", "pointwise-*gfx950.s"))
    if not paths:
        pytest.skip("no assembly here: the libraries were built elsewhere")
    with open(os.path.join(build.CSRC, "pointwise.hip")) as f:
        rule = re.search(r"^constexpr int waves_per_simd\(.*?^}$", f.read(), re.S | re.M)[0]
    with open(paths[0]) as f:
        found = {tuple(map(int, m[:5])): int(m[5]) for m in re.findall(
            r"\.name:\s+\S*pw_nchw_kernelILi(\d)ELb(\d)ELi1ELi([23])ELb(\d)ELb(\d)E\S*.*?\.vgpr_count:\s+(\d+)", f.read(), re.S)}
    assert len(found) == (4 + 1) * 2 * 2, found   # (codes of 32-bit accumulators have a kernel for whole ranges and one for others)
    source = tmp_path / "rule.cpp"
    source.write_text("#include <cstdio>\n" + rule + "\nint main() {\n" + "".join(
        f'  std::printf("%d\\n", waves_per_simd({mode}, {acc16}, {ch}, {small}));\n' for mode, acc16, ch, small, _ in found) + "}\n")
    subprocess.run(["g++", "-std=c++17", str(source), "-o", str(tmp_path / "rule")], check=True)
    counted = map(int, subprocess.run([str(tmp_path / "rule")], capture_output=True, text=True, check=True).stdout.split())
    assert dict(zip(found, counted)) == {k: REGISTERS // ((v + 7) // 8 * 8) for k, v in found.items()}
