"""CPU test of the row kernels' generated code: rotating a bf16 row in blocks of 2048 or 4096 elements, a block per wavefront, keeps
every value in registers (a spill goes to scratch memory, which every wavefront would reserve and some would use)."""
import os
import re
import subprocess

from paper_2501_02625_amd import _build


def test_long_blocks_stay_in_registers(tmp_path):
    asm = tmp_path / "row_transform.s"
    subprocess.run([_build._hipcc(), *_build.HIPCC_FLAGS, "--cuda-device-only", "-S",
                    os.path.join(_build.CSRC, "row_transform.hip"), "-o", str(asm)], check=True, capture_output=True)
    # row_transform_kernel<log2 of the segment, input type 0 = bf16, output type, log2 of the block, 0>
    kernels = re.findall(r"\.amdhsa_kernel \S*row_transform_kernelILi(1[12])ELi0ELi(\d)ELi\1ELi0EE.*?"
                         r"\.amdhsa_private_segment_fixed_size (\d+)", asm.read_text(), re.S)
    assert {k[:2] for k in kernels} == {("11", "0"), ("12", "0"), ("11", "3"), ("12", "3")}
    assert all(k[2] == "0" for k in kernels), kernels
