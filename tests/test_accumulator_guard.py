"""CPU test of the build's check on the INT8 GEMM's generated code (_build.accumulator_faults): the accumulators are registers
named in inline assembly, so the compiler must neither use one itself nor spill."""
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
