"""How the depthwise matrix kernel divides its row tiles, on the CPU (csrc/dw_split.h, which the launch includes too)."""
import os
import subprocess

from conftest import ROOT


def test_every_cu_has_its_share(tmp_path):
    exe = str(tmp_path / "dw_split")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2103_14949_amd", "csrc"),
                    os.path.join(ROOT, "tests", "dw_split_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "depthwise split: ok" in r.stdout, r.stdout + r.stderr
