"""Errors of the runtime, on the CPU: a refused call is reported by the entry point that made it, whichever of its calls it was,
and by no later one."""
import os
import subprocess

from conftest import ROOT
from paper_2103_14949_amd import build


def test_a_refused_call_is_reported_once(tmp_path):
    exe = str(tmp_path / "launch_status")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    lib = os.path.dirname(build.LIB)
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-isystem", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "launch_status_driver.cpp"), "-rdynamic",
                    build.LIB, f"-Wl,-rpath,{lib}", f"-Wl,-rpath-link,{rocm}/lib", f"-Wl,-rpath,{rocm}/lib", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "launch statuses: ok" in r.stdout, r.stdout[-4000:] + r.stderr
