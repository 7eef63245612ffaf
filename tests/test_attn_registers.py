"""Registers of attention kernels whose workgroups a compute unit can hold three of: the vector registers of a SIMD (512 per
lane) are shared by its waves, four waves to a workgroup, so three need at most 168 each (CPU only: compiled, not run)."""
import re
import subprocess

import pytest

from paper_2403_09919_amd import build as rd_build

KERNELS = """
#include "rd_tree_attn_mfma.h"
template __global__ void rd::rd_tree_attn_mfma_kernel<%(t)s, 64, 3, 4, false, true, false>(rd::AttnArgs);
template __global__ void rd::rd_tree_attn_mfma_kernel<%(t)s, 64, 3, 4, false, true, true>(rd::AttnArgs);
"""


@pytest.mark.parametrize("t", ["__bf16", "_Float16"])
def test_rotary_d64_keeps_three_workgroups(tmp_path, t):
    (tmp_path / "k.hip").write_text(KERNELS % {"t": t})
    subprocess.run(["/opt/rocm/bin/hipcc", *rd_build.FLAGS, "-w", "--cuda-device-only", "-S", "-I", rd_build.CSRC, "-I", rd_build.ROOT + "/include",
                    str(tmp_path / "k.hip"), "-o", str(tmp_path / "k.s")], check=True, capture_output=True)
    asm = (tmp_path / "k.s").read_text()
    assert [int(n) <= 512 // 3 // 8 * 8 for n in re.findall(r"\.vgpr_count:\s+(\d+)", asm)] == [True, True]
    assert re.findall(r"\.vgpr_spill_count:\s+(\d+)", asm) == ["0", "0"]
