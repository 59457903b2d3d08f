"""The offsets of the dense kernels' loads into LDS, on the CPU: no load reaches beyond its operand, for every place inside a
stage that a reduction can end at (csrc/stream_offset.h, which the kernel includes too)."""
import os
import subprocess

from conftest import ROOT


def test_every_load_is_inside_its_operand(tmp_path):
    exe = str(tmp_path / "stream_offsets")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2103_14949_amd", "csrc"),
                    os.path.join(ROOT, "tests", "stream_offset_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "stream offsets: ok" in r.stdout, r.stdout + r.stderr
