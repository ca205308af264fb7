"""Builds libhalo.so (hand-written HIP kernels for gfx950 + the C ABI) and the native half of the Python binding in-tree."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_PATH = os.path.join(PKG_DIR, "libhalo.so")
NATIVE_PATH = os.path.join(PKG_DIR, "_halo_native.so")
BUILD_DIR = os.path.join(PKG_DIR, "_build")

SOURCES = ["halo_api.hip", "row_transform.hip", "col_ops.hip", "gemm_i8.hip", "gemm_mx6.hip", "row_kron.hip", "lowrank.hip"]

# -ffp-contract=off: every fp32 add/mul of the rotation and the quantiser is rounded on its own, which is
# what makes the INT8 codes reproducible bit for bit.  Packed fp32 instructions are switched off.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I" + INCLUDE, "-I" + CSRC,
]


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: libhalo needs the ROCm toolchain to build")


def _run(cmd, cwd=None):
    proc = subprocess.run(cmd, capture_output=True, text=True, cwd=cwd)
    err = "\n".join(l for l in proc.stderr.splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if proc.returncode != 0:
        raise RuntimeError("build step failed: %s\n%s\n%s" % (" ".join(cmd), proc.stdout, err))
    return err


# Kernels whose accumulators are accumulation registers named in the text of inline assembly (csrc/matrix_asm.h), by source.
ACCUMULATOR_KERNELS = "gemm_i8_kernel"
ACCUMULATOR_SOURCES = {"gemm_i8.hip": ACCUMULATOR_KERNELS, "gemm_mx6.hip": "gemm_mx6_lines_kernel"}


def accumulator_faults(asm: str, kernel: str = ACCUMULATOR_KERNELS):
    """What the generated code of the kernels named `kernel` does to registers that the compiler does not know to be taken: uses
    of an accumulation register or of m0 outside inline assembly, and scratch memory (a spill could go to an accumulation
    register as well).  Returns (number of kernels looked at, list of faults)."""
    name = inline = None
    seen, faults = set(), []
    for line in asm.splitlines():
        label = re.match(r"(\w+):", line)
        if label and kernel in label.group(1):
            name, inline = label.group(1), False
            seen.add(name)
        elif name is None:
            continue
        elif line.startswith(".Lfunc_end"):
            name = None
        elif "#ASMSTART" in line:
            inline = True
        elif "#ASMEND" in line:
            inline = False
        elif not inline:
            code = line.split(";")[0]
            if re.match(r"\s*scratch_", code) or \
                    re.search(r"\ba(\d+|\[\d+(:\d+)?\])(?=[\s,]|$)|accvgpr|\bm0\b", code):
                faults.append("%s: %s" % (name, code.strip()))
            elif re.match(r"\s*\.amdhsa_private_segment_fixed_size\s+[1-9]", code):
                faults.append("%s: %s" % (name, code.strip()))
    return len(seen), faults


def _compile(src: str, obj: str) -> str:
    cmd = [_hipcc(), *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if src not in ACCUMULATOR_SOURCES:
        return _run(cmd)
    with tempfile.TemporaryDirectory() as tmp:
        log = _run(cmd + ["-save-temps"], cwd=tmp)
        with open(os.path.join(tmp, src.replace(".hip", "-hip-amdgcn-amd-amdhsa-gfx950.s"))) as f:
            count, faults = accumulator_faults(f.read(), ACCUMULATOR_SOURCES[src])
    if not count or faults:
        raise RuntimeError("%s: the compiler uses registers or scratch memory of %d kernels that hold their accumulators in "
                           "registers it does not know of:\n%s" % (src, count, "\n".join(faults[:20])))
    return log


def _build_native() -> str:
    """_halo_native.so: plain C++ against torch's headers, linked to libhalo.so next to it."""
    import torch
    tdir = os.path.dirname(torch.__file__)
    inc = os.path.join(tdir, "include")
    return _run([shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wno-attributes",
                 "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
                 "-I" + INCLUDE, "-I" + inc, "-I" + os.path.join(inc, "torch", "csrc", "api", "include"),
                 "-I" + sysconfig.get_paths()["include"],
                 os.path.join(CSRC, "native_binding.cpp"), "-o", NATIVE_PATH,
                 "-L" + os.path.join(tdir, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
                 "-L" + PKG_DIR, "-l:libhalo.so", "-Wl,-rpath,$ORIGIN"])


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link libhalo.so next to this file. Always recompiles."""
    hipcc = _hipcc()
    os.makedirs(BUILD_DIR, exist_ok=True)
    objs = [os.path.join(BUILD_DIR, s.replace(".hip", ".o")) for s in SOURCES]

    with ThreadPoolExecutor(max_workers=min(7, len(SOURCES))) as pool:
        logs = list(pool.map(_compile, SOURCES, objs))
    logs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH]))
    logs.append(_build_native())
    if verbose:
        for l in logs:
            if l.strip():
                print(l)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
