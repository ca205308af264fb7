"""CPU tests of the build's checks on the matrix kernels' generated code: the accumulators are registers named in inline assembly, so
the compiler must neither use one itself nor spill (_build.accumulator_faults), and LDS reads in inline assembly deliver their
registers at a later wait (_build.outstanding_read_faults)."""
import os
import subprocess

import pytest

from paper_2501_02625_amd import _build

KERNEL = """_ZN4halo14gemm_i8_kernelILi8EEEv:
\ts_load_dwordx2 s[0:1], s[4:5], 0x0
\t;;#ASMSTART
\tv_mfma_i32_16x16x64_i8 a[0:3], v[0:3], v[4:7], a[0:3]
\t;;#ASMEND
\t;;#ASMSTART
\ts_mov_b32 m0, s3
\ts_nop 0
\tbuffer_load_dwordx4 v1, s[8:11], 0 offen lds
\t;;#ASMEND
\tglobal_store_dword v[0:1], v2, off ; a note on a12
%s
\ts_endpgm
\t.amdhsa_kernel _ZN4halo14gemm_i8_kernelILi8EEEv
\t\t.amdhsa_private_segment_fixed_size %d
\t.end_amdhsa_kernel
.Lfunc_end0:
_ZN4halo20gemm_i8_small_kernelILi1EEEv:
\tv_mfma_i32_16x16x64_i8 a[0:3], v[0:3], v[4:7], a[0:3]
.Lfunc_end1:
"""


@pytest.mark.parametrize("line,scratch,clean", [
    ("\tv_mov_b32_e32 v3, v4", 0, True),
    ("\tv_accvgpr_write_b32 a255, v3", 0, False),
    ("\tv_mov_b32_e32 v3, a12", 0, False),
    ("\tglobal_load_dwordx4 a[8:11], v[0:1], off", 0, False),
    ("\tscratch_store_dword off, v3, off", 0, False),
    ("\ts_mov_b32 m0, s7", 0, False),
    ("\tv_mov_b32_e32 v3, v4", 16, False),
])
def test_uses_outside_inline_assembly_are_found(line, scratch, clean):
    count, faults = _build.accumulator_faults(KERNEL % (line, scratch))
    assert count == 1 and (faults == []) == clean, faults


READS = """_ZN4halo1kEv:
%s
\ts_endpgm
.Lfunc_end0:
"""


def inline(text):
    return "\t;;#ASMSTART\n" + text + "\n\t;;#ASMEND\n"


READ = inline("\tds_read_b128 v[8:11], v2 offset:16")
LATER = inline("\tds_read_b64 v[12:13], v2")
WAIT = inline("\ts_waitcnt vmcnt(3) lgkmcnt(%d)")


@pytest.mark.parametrize("text,clean", [
    (READ + "\tv_mov_b32_e32 v7, v12\n" + WAIT % 0 + "\tv_mov_b32_e32 v8, v7", True),
    (READ + "\tv_mov_b32_e32 v10, v7", False),                                # free for the compiler, and overwritten later
    (READ + "\tv_mov_b32_e32 v7, v11", False),                                # not there yet
    (READ + inline("\tv_mfma_i32_16x16x64_i8 a[0:3], v[4:7], v[8:11], a[0:3]"), False),
    (READ + READ + WAIT % 0 + "\tv_mov_b32_e32 v10, v7", True),               # two reads of one register arrive in order
    (READ + inline("\tds_read_b64 v[12:13], v8"), False),                     # but an address has to be there
    (READ + LATER + WAIT % 1 + "\tv_mov_b32_e32 v8, v7", True),
    (READ + LATER + WAIT % 1 + "\tv_mov_b32_e32 v13, v7", False),
    (READ + "\tds_write_b32 v1, v3\n" + WAIT % 1 + "\tv_mov_b32_e32 v8, v7", True),
    (READ + "\tds_bpermute_b32 v20, v1, v3\n\ts_waitcnt vmcnt(0)\n\tv_mov_b32_e32 v8, v7", False),
    # around a loop; out of it on one of two ways; past a wait that only one of two ways has
    (".LBB0_1:\n" + WAIT % 1 + "\tv_mov_b32_e32 v12, v7\n" + READ + LATER + "\ts_cbranch_scc1 .LBB0_1\n" + WAIT % 0, False),
    (".LBB0_1:\n" + WAIT % 0 + "\tv_mov_b32_e32 v12, v7\n" + READ + LATER + "\ts_cbranch_scc1 .LBB0_1\n" + WAIT % 0, True),
    (READ + "\ts_cbranch_scc1 .LBB0_2\n" + WAIT % 0 + ".LBB0_2:\n\tv_mov_b32_e32 v8, v7", False),
    (READ + "\ts_branch .LBB0_2\n\tv_mov_b32_e32 v8, v7\n.LBB0_2:\n" + WAIT % 0, True),
    (READ + ".LBB0_3:\n\ts_cbranch_execnz .LBB0_2\n\tv_mov_b32_e32 v8, v7\n.LBB0_2:\n" + WAIT % 0, True),
])
def test_reads_that_nothing_has_waited_for_are_found(text, clean):
    count, faults = _build.outstanding_read_faults(READS % text)
    assert count == 1 and (faults == []) == clean, faults


@pytest.mark.parametrize("source", sorted(_build.ACCUMULATOR_SOURCES))
def test_matrix_kernels_wait_for_their_reads(source, tmp_path):
    """No register of a fragment is used, or used for something else, before its read has been waited for: the last unit of K
    reads fragments that nothing uses."""
    asm = tmp_path / "kernels.s"
    subprocess.run([_build._hipcc(), *_build.HIPCC_FLAGS, "--cuda-device-only", "-S", os.path.join(_build.CSRC, source), "-o", str(asm)],
                   check=True, capture_output=True)
    count, faults = _build.outstanding_read_faults(asm.read_text())
    assert count and not faults, faults
