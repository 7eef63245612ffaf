"""The 16-byte write-through store that carries partial results between workgroups, as compiled for gfx950: the wait states
around it are those the compiler keeps around a 16-byte store of its own (CPU only: compiled, not run)."""
import re
import subprocess

from paper_2403_09919_amd import build as rd_build

SOURCE = """
#include "rd_internal.h"
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
// a matrix result is stored, and the registers it was stored from are written at once
#define KERNEL(name, store)                                                                       \\
    extern "C" __global__ void name(float *out, const bf16x8 *in)                                 \\
    {                                                                                             \\
        const bf16x8 a = in[threadIdx.x], b = in[threadIdx.x + 64];                               \\
        f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0); \\
        float *p = out + threadIdx.x * 4;                                                         \\
        store;                                                                                    \\
        asm volatile("v_add_f32 %0, 1.0, %0" : "+v"(c[0]));                                       \\
        out[threadIdx.x + 4096] = c[0];                                                           \\
    }
KERNEL(known_store, *reinterpret_cast<f32x4 *>(p) = c)
KERNEL(device_store, rd::st_dev4(p, c[0], c[1], c[2], c[3]))
"""


def _wait_states(lines):
    """Wait states that the instructions of `lines` take: one each, s_nop n + 1."""
    n = 0
    for line in lines:
        m = re.match(r"s_nop (\d+)", line)
        n += int(m.group(1)) + 1 if m else 1
    return n


def _around_store(asm, kernel):
    """Wait states between the matrix instruction and the 16-byte store, and between that and the write of its data."""
    body = asm[asm.index("\n%s:" % kernel):]
    code = [l.strip() for l in body[:body.index("s_endpgm")].splitlines()]
    code = [l for l in code if re.match(r"[a-z]+_", l)]
    mfma = next(i for i, l in enumerate(code) if l.startswith("v_mfma"))
    store = next(i for i, l in enumerate(code) if l.startswith("global_store_dwordx4"))
    write = next(i for i, l in enumerate(code) if l.startswith("v_add_f32"))
    assert mfma < store < write
    return code[store], _wait_states(code[mfma + 1:store]), _wait_states(code[store + 1:write])


def test_wait_states_around_the_16_byte_store(tmp_path):
    src, out = tmp_path / "store.hip", tmp_path / "store.s"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", *rd_build.FLAGS, "-w", "--cuda-device-only", "-S", "-I", rd_build.CSRC,
                    "-I", rd_build.ROOT + "/include", str(src), "-o", str(out)], check=True, capture_output=True)
    asm = out.read_text()
    _, before, after = _around_store(asm, "known_store")
    assert before >= 8 and after >= 2
    store, got_before, got_after = _around_store(asm, "device_store")
    assert re.search(r"\bsc1$", store)               # written through the XCD's L2
    assert got_before >= before and got_after >= after
