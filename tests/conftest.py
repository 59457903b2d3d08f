import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

GOLDEN = os.path.join(ROOT, "tests", "golden")


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def read_golden(name):
    """Rows of whitespace-separated tokens; '#' starts a comment."""
    rows = []
    with open(os.path.join(GOLDEN, name)) as f:
        for line in f:
            line = line.split("#", 1)[0].strip()
            if line:
                rows.append(line.split())
    return rows


@pytest.fixture(scope="session")
def ref():
    from oracle import hago_ref
    hago_ref.build()
    hago_ref.lib()
    return hago_ref


def build_against_fake_runtime(source, exe):
    """A program that loads the library as built and stands in for the HIP runtime (tests/fake_runtime.h)."""
    import subprocess
    from paper_2103_14949_amd import build
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-isystem", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", source), "-rdynamic", build.LIB,
                    f"-Wl,-rpath,{os.path.dirname(build.LIB)}", f"-Wl,-rpath-link,{rocm}/lib", f"-Wl,-rpath,{rocm}/lib", "-o", exe], check=True)


@pytest.fixture(scope="session")
def routes(tmp_path_factory):
    """Calls (lines of tests/routes_driver.cpp) -> the kernels that serve each, on the CPU."""
    import subprocess
    exe = str(tmp_path_factory.mktemp("routes") / "routes")
    build_against_fake_runtime("routes_driver.cpp", exe)

    def kernels(calls):
        r = subprocess.run([exe], input="".join(c + "\n" for c in calls), capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [[re.sub(r"^void |hago::|\(anonymous namespace\)::|\(.*$| ", "", k.split("(", 2)[0] + k.split(")::", 1)[1]) for k in line.split("\t")[:-1]]
                for line in r.stdout.splitlines()]
    return kernels


@pytest.fixture(params=["plain", "ws", "ws_stream"])
def conv_entry(request):
    """Runs a convolution parity test once per entry point (see gpu_util.qconv2d); "ws_stream" also
    switches off the kernels specialised for 1x1 and 3x3 geometries, so that the streaming implicit
    GEMM over the workspace copies meets every geometry."""
    import gpu_util
    import paper_2103_14949_amd as hago
    gpu_util.CONV_ENTRY["name"] = "plain" if request.param == "plain" else "ws"
    if request.param == "ws_stream":
        hago.set_test_hook(hago.HOOK_GEMM_PATH, 2)
    yield request.param
    hago.set_test_hook(hago.HOOK_GEMM_PATH, 0)
    gpu_util.CONV_ENTRY["name"] = "plain"


@pytest.fixture
def stream_tile():
    """Forces a tile shape of the streaming dense kernel for the rest of a test."""
    import paper_2103_14949_amd as hago
    yield lambda tile: hago.set_test_hook(hago.HOOK_STREAM_TILE, tile)
    hago.set_test_hook(hago.HOOK_STREAM_TILE, -1)


@pytest.fixture
def gemm_path():
    """Forces the GEMM kernel family (1: general register-staged, 2: streaming without the kernels
    specialised for 1x1 and 3x3 convolutions) for the rest of a test."""
    import paper_2103_14949_amd as hago
    yield lambda path: hago.set_test_hook(hago.HOOK_GEMM_PATH, path)
    hago.set_test_hook(hago.HOOK_GEMM_PATH, 0)
