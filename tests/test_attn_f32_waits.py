"""What a wave of the fp32 attention kernel waits for before the workgroup first meets (CPU only: compiled, not run): Q alone,
with the loads of its first tile of K and V still under way."""
import os
import re
import subprocess

from paper_2403_09919_amd import build as rd_build


def test_first_barrier_waits_for_q_alone(tmp_path):
    subprocess.run(["/opt/rocm/bin/hipcc", *rd_build.FLAGS, "-w", "--cuda-device-only", "-S", "-I", rd_build.CSRC, "-I", rd_build.ROOT + "/include",
                    os.path.join(rd_build.CSRC, "rd_tree_attn_f32.hip"), "-o", str(tmp_path / "k.s")], check=True, capture_output=True)
    kernels = re.findall(r"^(_ZN\w*rd_tree_attn_f32_kernelILi(\d+)E\w*):(.*?)^\.Lfunc_end", (tmp_path / "k.s").read_text(), re.M | re.S)
    assert {int(D) for _, D, _ in kernels} == {64, 128}
    for name, D, code in kernels:
        waits = re.findall(r"s_waitcnt[^\n]*vmcnt\((\d+)\)", code[:code.index("s_barrier")])
        tile = int(D) // 16 + 4 * (int(D) // 64)             # 16-byte loads of K and V
        assert waits and int(waits[-1]) >= tile, (name, waits)
