"""Errors of the runtime, on the CPU: a refused call is reported by the entry point that made it, whichever of its calls it was,
and by no later one."""
import subprocess

from conftest import build_against_fake_runtime


def test_a_refused_call_is_reported_once(tmp_path):
    exe = str(tmp_path / "launch_status")
    build_against_fake_runtime("launch_status_driver.cpp", exe)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "launch statuses: ok" in r.stdout, r.stdout[-4000:] + r.stderr
