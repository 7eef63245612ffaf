"""Memory instructions around which the compiler keeps wait states only if it knows them, as compiled for gfx950 (CPU only:
compiled, not run): the 16-byte write-through store that carries partial results between workgroups, and the copies into LDS."""
import re
import subprocess

import pytest

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
// a base that a vector instruction hands over in scalar registers
extern "C" __global__ void known_scalar(float *out, const int *at)
{
    auto rsrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, -1, 0x00027000);
    const int base = __builtin_amdgcn_readfirstlane(at[threadIdx.x]);
    out[threadIdx.x] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)threadIdx.x * 4, base, 0));
}
#define COPY(name, copy, bytes)                                                                   \
    extern "C" __global__ void name(float *out, const uintptr_t *at)                              \
    {                                                                                             \
        __shared__ __attribute__((aligned(16))) float s[256];                                     \
        typedef __attribute__((address_space(3))) float lds_float;                                \
        rd::copy(at[threadIdx.x], threadIdx.x * bytes, (uint32_t)(uintptr_t)(lds_float *)s);      \
        rd::wait_vm<0>();                                                                         \
        out[threadIdx.x] = s[threadIdx.x];                                                        \
    }
COPY(copy_16, dma16, 16)
COPY(copy_4, dma4, 4)
"""


def _wait_states(lines):
    """Wait states that the instructions of `lines` take: one each, s_nop n + 1."""
    n = 0
    for line in lines:
        m = re.match(r"s_nop (\d+)", line)
        n += int(m.group(1)) + 1 if m else 1
    return n


def _code(asm, kernel):
    body = asm[asm.index("\n%s:" % kernel):]
    code = [l.strip() for l in body[:body.index("s_endpgm")].splitlines()]
    return [l for l in code if re.match(r"[a-z]+_", l)]


def _scalars(operands):
    """Numbers of the scalar registers that are named."""
    found = {int(n) for n in re.findall(r"\bs(\d+)\b", operands)}
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", operands):
        found |= set(range(int(a), int(b) + 1))
    return found


def _around_store(asm, kernel):
    """Wait states between the matrix instruction and the 16-byte store, and between that and the write of its data."""
    code = _code(asm, kernel)
    mfma = next(i for i, l in enumerate(code) if l.startswith("v_mfma"))
    store = next(i for i, l in enumerate(code) if l.startswith("global_store_dwordx4"))
    write = next(i for i, l in enumerate(code) if l.startswith("v_add_f32"))
    assert mfma < store < write
    return code[store], _wait_states(code[mfma + 1:store]), _wait_states(code[store + 1:write])


def _behind_scalar(asm, kernel, load):
    """Wait states between the load and the last vector instruction before it that writes one of the scalar registers it reads
    (none: None; a scalar instruction waits for what it reads, and its results may be used at once)."""
    code = _code(asm, kernel)
    at = next(i for i, l in enumerate(code) if l.startswith(load))
    read = _scalars(code[at].split(None, 1)[1])
    for i in range(at - 1, -1, -1):
        wrote = _scalars(code[i].split(None, 1)[1].split(",")[0]) & read if " " in code[i] else set()
        if wrote and code[i].startswith("v_"):
            return _wait_states(code[i + 1:at])
        read -= wrote
    return None


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    d = tmp_path_factory.mktemp("wait_states")
    (d / "k.hip").write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", *rd_build.FLAGS, "-w", "--cuda-device-only", "-S", "-I", rd_build.CSRC,
                    "-I", rd_build.ROOT + "/include", str(d / "k.hip"), "-o", str(d / "k.s")], check=True, capture_output=True)
    return (d / "k.s").read_text()


def test_around_the_16_byte_store(asm):
    _, before, after = _around_store(asm, "known_store")
    assert before >= 8 and after >= 2
    store, got_before, got_after = _around_store(asm, "device_store")
    assert re.search(r"\bsc1$", store)               # written through the XCD's L2
    assert got_before >= before and got_after >= after


@pytest.mark.parametrize("kernel,load", [("copy_16", "global_load_lds_dwordx4"), ("copy_4", "global_load_lds_dword")])
def test_in_front_of_copies_into_lds(asm, kernel, load):
    need = _behind_scalar(asm, "known_scalar", "buffer_load_dword")
    assert need >= 5
    got = _behind_scalar(asm, kernel, load)
    assert got is None or got >= need
