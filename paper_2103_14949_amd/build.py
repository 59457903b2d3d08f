"""Build libhago.so (the C-ABI library) from the HIP sources for gfx950, and the binding's native
marshalling module (_native.so, host code against torch's headers).

hipcc cross-compiles without a GPU.  The libraries are written next to this file
so that they travel with the source tree.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhago.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC",
    "-ffp-contract=off",                       # simquant: no fused multiply-add
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-mllvm", "-amdgpu-kernarg-preload-count=14",   # leading scalar arguments are in registers when a wavefront starts
    "-save-temps=obj",                         # the assembly, for check_assembly
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


NATIVE_LIB = os.path.join(HERE, "_native.so")


def build_native(verbose: bool = False) -> str:
    """Compile the binding's native module; always recompiles."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    include = [*cpp_extension.include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           *[f"-isystem{d}" for d in include], os.path.join(CSRC, "native.cpp"), "-o", NATIVE_LIB, f"-L{torch_lib}",
           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", f"-Wl,-rpath,{torch_lib}"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return NATIVE_LIB


def check_shift_amounts(assembly: str) -> list[str]:
    """The kernels that hold a 64-bit shift with its amount in the last register allocated to a wavefront
    (registers come in blocks of eight), which this GPU gets wrong now and then; see HAGO_SPARE_REGISTER."""
    found, shifts, kernel, label = [], {}, None, None
    for line in assembly.splitlines():
        if m := re.match(r"(\w+):", line):
            label = m[1]
        elif m := re.match(r"\s+v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\w*\s+v\[\d+:\d+\], v(\d+),", line):
            # (local labels start with ".L" and do not match; a function's own label is the last one seen)
            shifts.setdefault(label, []).append((int(m[1]), line.strip()))
        elif m := re.match(r"\s+\.amdhsa_kernel (\S+)", line):
            kernel = m[1]
        elif m := re.match(r"\s+\.amdhsa_next_free_vgpr (\d+)", line):
            last = (int(m[1]) + 7) // 8 * 8 - 1
            found += [f"{kernel}: {text}" for amount, text in shifts.get(kernel, []) if amount == last]
    return found


def check_lds_loads(assembly: str) -> list[str]:
    """Loads into the LDS that directly follow a write of m0, which they take their address from: one wait state is
    required between the two, and in inline assembly nobody inserts it."""
    return [f"{m[1].strip()}; {m[2].strip()}" for m in
            re.finditer(r"^\s+(s_\w+\s+m0,.*)\n(?:\s*;.*\n)*\s+((?:buffer|global|scratch)_load_\w+.*\blds\b.*|global_load_lds_.*)$",
                        assembly, re.M)]


def check_wide_stores(assembly: str) -> list[str]:
    """Stores of more than eight bytes in inline assembly that are not followed by two wait states: the registers of their data
    must not be written before, and nobody inserts them there."""
    found = []
    for block in re.findall(r";;?#ASMSTART\n(.*?);;?#ASMEND", assembly, re.S):
        for m in re.finditer(r"^\s*((?:global|buffer|flat|scratch)_store_dwordx[34]\b.*)\n(.*)", block, re.M):
            nop = re.match(r"\s*s_nop (\d+)", m[2])
            if not nop or int(nop[1]) < 1:
                found.append(m[1].strip())
    return found


def check_lane_exchanges(assembly: str) -> list[str]:
    """Results of vector instructions in inline assembly that lanes exchange (DPP, permlane) fewer than two wait states later, on any
    way there: those read what stands in the registers before it, and behind inline assembly nobody inserts the wait states."""
    def registers(text):
        return {n for first, last in re.findall(r"\bv\[?(\d+)(?::(\d+)\])?", text) for n in range(int(first), int(last or first) + 1)}

    instructions, labels, inside = [], {}, False   # (text, in inline assembly)
    for line in assembly.splitlines():
        if "ASMSTART" in line or "ASMEND" in line:
            inside = "ASMSTART" in line
        elif m := re.match(r"([\w.$]+):", line):
            labels[m[1]] = len(instructions)
        elif m := re.match(r"\s+([a-z]\w+(?: .*?)?)\s*(?:;.*)?$", line):
            instructions.append((m[1], inside))
    found = []
    for at, (text, inside) in enumerate(instructions):
        if not inside or not text.startswith("v_"):
            continue
        written = registers(text.split(",")[0])
        ways, seen = [(at + 1, 0)], set()
        while ways:
            i, states = ways.pop()
            if states >= 2 or i >= len(instructions) or (i, states) in seen:
                continue
            seen.add((i, states))
            later = instructions[i][0]
            # (a permlane swap reads both its registers; a DPP instruction all but its first, unless that keeps some of its bits)
            if later.startswith("v_permlane") and registers(later) & written or (
                    re.search(r"_dpp\b|\b(?:quad_perm|row_\w+|wave_\w+)\b", later) and registers(later.split(",", 1)[-1]) & written):
                found.append(f"{text}; {later}")
            m = re.match(r"s_(c?branch)\w*\s+(\S+)", later)
            if m and m[2] in labels:
                ways.append((labels[m[2]], states + 1))
            if not m or m[1] == "cbranch":
                nop = re.match(r"s_nop (\w+)", later)
                ways.append((i + 1, states + (int(nop[1], 0) + 1 if nop else 1)))
    return found


def check_assembly(assembly: str) -> list[str]:
    """What the kernels must not hold, and the compiler does not avoid."""
    return ([f"64-bit shift by the last allocated register (add HAGO_SPARE_REGISTER): {f}" for f in check_shift_amounts(assembly)] +
            [f"wide store without two wait states behind it: {f}" for f in check_wide_stores(assembly)] +
            [f"lane exchange without two wait states behind inline assembly: {f}" for f in check_lane_exchanges(assembly)] +
            [f"LDS load without a wait state after m0: {f}" for f in check_lds_loads(assembly)])


def _check_assembly(directory):
    found = []
    for path in sorted(glob.glob(os.path.join(directory, "*gfx950.s"))):
        with open(path) as f:
            found += check_assembly(f.read())
    if found:
        raise RuntimeError("\n".join(found))


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every .hip file and link the shared library, and the native module; always recompiles."""
    build_native(verbose)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, os.path.basename(src) + ".o") for src in sources()]

    def compile_one(src, obj):
        cmd = [hipcc, *HIPCC_FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        _drain([(src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))], verbose)

    # first, so that none of them is waited for alone
    slow = ("qgemm_dma_other.hip", "qgemm_line_other.hip", "qgemm_dma.hip", "qgemm_dma_clipped.hip", "conv_gather.hip", "dwconv.hip")
    with concurrent.futures.ThreadPoolExecutor(jobs) as pool:
        list(pool.map(lambda so: compile_one(*so), sorted(zip(sources(), objs), key=lambda so: not so[0].endswith(slow))))
    _check_assembly(objdir)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    subprocess.run(cmd, check=True)
    return LIB


def _drain(procs, verbose):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        # the host pass does not know the packed-fp32 target feature and says so
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l]
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n" + "\n".join(lines))
        if verbose and lines:
            print("\n".join(lines), flush=True)


PHASE_LIB = os.path.join(HERE, "libhago_phase.so")


def build_phase_timing(verbose: bool = False) -> str:
    """Development variant of the library for `bench.py --phase-stamps`: the GEMM kernels write a
    timestamp per workgroup at each phase boundary (first loads, main loop, channel terms,
    requantize, copy-out).  Needs the objects of a normal build() for the other sources."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build", "phase")
    os.makedirs(objdir, exist_ok=True)
    timed = [kernel + results for kernel in ("qgemm_dma", "qgemm_line") for results in (".hip", "_clipped.hip", "_other.hip")] + ["qgemm.hip"]
    procs, objs = [], []
    for src in sources():
        base = os.path.basename(src)
        if base in timed:
            obj = os.path.join(objdir, base + ".o")
            cmd = [hipcc, *HIPCC_FLAGS, "-DHAGO_PHASE_TIMING", "-c", src, "-o", obj]
            procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        else:
            obj = os.path.join(HERE, "_build", base + ".o")
            if not os.path.exists(obj):
                raise RuntimeError(f"{obj} is missing: run build() first")
        objs.append(obj)
    _drain(procs, verbose)
    _check_assembly(objdir)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", PHASE_LIB], check=True)
    return PHASE_LIB


if __name__ == "__main__":
    if "--phase-timing" in sys.argv:
        print(build_phase_timing(verbose="-v" in sys.argv))
    else:
        print(build(verbose="-v" in sys.argv))
