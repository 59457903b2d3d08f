"""How the elementwise kernels divide channel-last and ragged tensors, on the CPU (csrc/span_split.h, which the launches include too)."""
import os
import subprocess

from conftest import ROOT


def test_every_operator_has_its_lanes(tmp_path):
    exe = str(tmp_path / "span_split")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2103_14949_amd", "csrc"),
                    os.path.join(ROOT, "tests", "span_split_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "span split: ok" in r.stdout, r.stdout + r.stderr
