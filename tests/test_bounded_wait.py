"""The wait of the last workgroup for a word whose store is on its way ends whether or not the word comes (CPU only: the wait
is run on the host with a word that never changes), and no kernel waits for memory in any other way."""
import os
import re
import subprocess

from paper_2403_09919_amd import build as rd_build

SOURCE = """
#include "rd_internal.h"
#include <stdio.h>
int main()
{
    long reads = 0;
    const unsigned never = rd::poll([&]() { ++reads; return 7u; }, [](unsigned x) { return x == 0; });
    printf("%u %ld\\n", never, reads);
    reads = 0;
    const unsigned third = rd::poll([&]() { return (unsigned)++reads; }, [](unsigned x) { return x == 3; });
    printf("%u %ld\\n", third, reads);
    return 0;
}
"""


def test_a_word_that_never_comes_ends_the_wait(tmp_path):
    (tmp_path / "poll.hip").write_text(SOURCE)
    exe = tmp_path / "poll"
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-std=c++17", "-O1", "-w", "-I", rd_build.CSRC, "-I", rd_build.ROOT + "/include",
                    str(tmp_path / "poll.hip"), "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split()
    assert out[0] == "7" and 1000 <= int(out[1]) <= 1 << 20      # generous, and an end
    assert out[2:] == ["3", "3"]


def test_no_loop_on_a_memory_word_without_an_end():
    """Loops whose condition or body reads a word past the caches (ld_dev, device-scope atomic loads) go through rd::poll."""
    for name in sorted(os.listdir(rd_build.CSRC)):
        with open(os.path.join(rd_build.CSRC, name)) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for loop in re.findall(r"\bdo\b[^;]*;\s*while\s*\([^;]*;|\bwhile\s*\([^;{]*[;{]", text):
            assert "ld_dev" not in loop and "__hip_atomic_load" not in loop, (name, loop)
