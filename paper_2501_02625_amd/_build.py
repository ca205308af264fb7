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


def _vector_registers(operands: str):
    """Numbers of the vector registers that the operands name."""
    regs = set()
    for lo, hi, one in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", operands):
        regs.update(range(int(lo), int(hi) + 1) if lo else (int(one),))
    return frozenset(regs)


def _blocks_of_kernels(asm: str):
    """Yields (kernel, blocks) for every kernel whose inline assembly reads LDS.  blocks: basic blocks in the order of the text, each
    (labels, instructions, jump target or None, falls through to the next?); an instruction is (text, inline?)."""
    name = None
    for line in asm.splitlines():
        code = line.split(";")[0].strip()
        label = re.match(r"([.\w$]+):", line)
        if label and not label.group(1).startswith(".L"):
            name, blocks, reads = label.group(1), [([], [], None, True)], False
            inline = False
        elif name is None:
            continue
        elif line.startswith(".Lfunc_end"):
            if reads:
                yield name, blocks
            name = None
        elif label:
            if blocks[-1][1]:
                blocks.append(([], [], None, True))
            blocks[-1][0].append(label.group(1))
        elif "#ASMSTART" in line:
            inline = True
        elif "#ASMEND" in line:
            inline = False
        elif code and not code.startswith("."):
            labels, instructions, _, _ = blocks[-1]
            instructions.append((code, inline))
            reads = reads or (inline and code.startswith("ds_read"))
            jump = re.match(r"s_(c?)branch\w*\s+(\S+)", code)
            if jump or code.startswith(("s_endpgm", "s_setpc")):
                # a block that is nothing but "jump if there is an active lane": entered with all of them, left by the jump
                falls = bool(jump and jump.group(1)) and not (code.startswith("s_cbranch_execnz") and len(instructions) == 1)
                blocks[-1] = (labels, instructions, jump and jump.group(2), falls)
                blocks.append(([], [], None, True))


def outstanding_read_faults(asm: str):
    """LDS reads written in inline assembly deliver their registers at a later wait, but the compiler takes them as written at once,
    and as free once nothing uses them.  Returns (number of kernels with such reads, list of faults): instructions that touch the
    destination of a read for which, on some way there, nothing has waited.  (Another read into the same registers is none: reads
    of one wavefront arrive in order.)"""
    seen, faults = set(), set()
    limit = 63                                # reads that a state keeps apart, newest first; older ones are taken together
    for name, blocks in _blocks_of_kernels(asm):
        seen.add(name)
        where = {label: n for n, block in enumerate(blocks) for label in block[0]}
        before = {0: ()}                      # block -> LDS instructions on their way at its start: the registers each one brings
        todo = [0]
        while todo:
            n = todo.pop()
            _, instructions, target, falls = blocks[n]
            flying = list(before[n])
            for code, inline in instructions:
                mnemonic, _, operands = code.partition(" ") if " " in code else code.partition("\t")
                operands = operands.strip()
                if mnemonic == "s_waitcnt":
                    count = re.search(r"lgkmcnt\((\d+)\)", operands)
                    if count:
                        del flying[int(count.group(1)):]
                    continue
                read = inline and mnemonic.startswith("ds_read")
                dest, _, rest = operands.partition(",")
                touched = _vector_registers(rest if read else operands)
                for regs in flying:
                    if regs & touched:
                        faults.add("%s: %s" % (name, code))
                if mnemonic.startswith("ds_"):
                    flying.insert(0, _vector_registers(dest) if read else frozenset())
                    if len(flying) > limit:
                        flying[limit - 1:] = [frozenset().union(*flying[limit - 1:])]
            for m in ([where[target]] if target in where else []) + ([n + 1] if falls and n + 1 < len(blocks) else []):
                old = before.get(m)
                if old is None:
                    new = tuple(flying)
                else:
                    size = max(len(old), len(flying))
                    pad = lambda state: list(state) + [frozenset()] * (size - len(state))
                    new = tuple(a | b for a, b in zip(pad(old), pad(flying)))
                if new != old:
                    before[m] = new
                    todo.append(m)
    return len(seen), sorted(faults)


def _compile(src: str, obj: str) -> str:
    cmd = [_hipcc(), *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if src not in ACCUMULATOR_SOURCES:
        return _run(cmd)
    with tempfile.TemporaryDirectory() as tmp:
        log = _run(cmd + ["-save-temps"], cwd=tmp)
        with open(os.path.join(tmp, src.replace(".hip", "-hip-amdgcn-amd-amdhsa-gfx950.s"))) as f:
            asm = f.read()
    count, faults = accumulator_faults(asm, ACCUMULATOR_SOURCES[src])
    if not count or faults:
        raise RuntimeError("%s: the compiler uses registers or scratch memory of %d kernels that hold their accumulators in "
                           "registers it does not know of:\n%s" % (src, count, "\n".join(faults[:20])))
    count, faults = outstanding_read_faults(asm)
    if not count or faults:
        raise RuntimeError("%s: in %d kernels that read LDS in inline assembly, instructions touch registers that a read has yet "
                           "to deliver:\n%s" % (src, count, "\n".join(faults[:20])))
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
