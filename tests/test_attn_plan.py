"""Launch plans of the attention kernels (csrc/rd_attn_common.h), on the CPU: a small program that prints them is
compiled against the header, host pass only."""
import os
import subprocess

import pytest

import attn_dealing

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "rd_attn_common.h"
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
using namespace rd;

// With arguments (B H N D C) the way the launch deals its workgroups.  Else one line per plan that breaks a rule; the last line
// counts the plans looked at.
int main(int argc, char **argv)
{
    if (argc > 5) {
        const AttnPlan p = attn_plan_make(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]));
        puts(p.n_rg > 1 && p.S == 1 ? "in turn" : p.sorted ? "ranked" : p.n_rg > 1 ? "places" : "heads");
        return 0;
    }
    const int ctxs[] = {0, 1, 32, 100, 300, 700, 1000, 1400, 1500, 2048, 3000, 5000, 9000, 20000, 40000, 131072};
    const int shapes[][2] = {{1, 1}, {1, 4}, {1, 5}, {1, 32}, {2, 40}, {4, 32}, {8, 32}, {3, 26}, {16, 52}, {24, 32}, {70, 3}, {300, 8}, {2048, 4}};
    long n = 0;
    for (int f32 = 0; f32 < 2; ++f32)
        for (int D = 64; D <= 128; D += 64)
            for (auto &s : shapes)
                for (int N = 1; N <= RD_MAX_N; ++N) {
                    size_t first = 0;
                    for (int C : ctxs) {
                        const AttnPlan p = attn_plan(s[0], s[1], N, D, C, f32 != 0);
                        const long long BH = (long long)s[0] * s[1];
                        const size_t part = (size_t)p.rg_tiles * 16 * (2 + D) * sizeof(float);
                        auto bad = [&](const char *what) { printf("B=%d H=%d N=%d D=%d C=%d f32=%d: %s\n", s[0], s[1], N, D, C, f32, what); };
                        if (C == ctxs[0]) first = p.counters_bytes;
                        if (p.counters_bytes != first) bad("the counters' place depends on the context");
                        if (p.counters_bytes < (size_t)BH * p.n_rg * sizeof(unsigned long long)) bad("counters overlap the partial results");
                        int most = 1;              // key ranges; one is written out directly
                        for (int g = 1; !f32 && g <= p.n_rg; ++g) {
                            const int own = attn_ranges(p.ranges, g), R = own > p.usual ? own : p.usual;
                            most = R > most ? R : most;
                            if (own < 1 || p.usual < 1 || (s[0] > kOneStep && own != p.usual)) bad("key ranges");
                            if (s[0] > 1 && own > p.usual && (BH + 7) / 8 * 8 * g * own > (p.waves == 8 ? 256 : 512)) bad("ranges that wait for a place");
                            if (R < 1 || (p.S > 1 ? R * g > p.S : R > 1)) bad("key ranges without workgroups");
                        }
                        const bool partials = f32 ? p.S > 1 : most > 1;
                        if (partials && p.total_bytes < p.counters_bytes + (size_t)BH * p.S * part) bad("no room for the partial results");
                        if (!f32 && !partials && p.total_bytes != p.counters_bytes) bad("room for partial results that nothing writes");
                        if (p.rg_tiles * p.n_rg * 16 < N) bad("rows without a group");
                        if ((p.S < p.n_rg && (f32 || p.S != 1)) || p.ranges == 0 || (p.waves != 4 && p.waves != 8)) bad("workgroups");
                        // kept plans: the one just made, and one that may have been pushed out since
                        for (int other : {C, ctxs[0], 300}) {
                            const AttnPlan kept = attn_plan(s[0], s[1], N, D, other, f32 != 0);
                            const AttnPlan made = f32 ? attn_plan_make_f32(s[0], s[1], N, D, other) : attn_plan_make(s[0], s[1], N, D, other);
                            if (memcmp(&kept, &made, sizeof(kept)) != 0) bad("a kept plan is not the one of these arguments");
                        }
                        const AttnPlan all = N % 7 ? p : f32 ? attn_plan_make_f32(s[0], s[1], N, D, C, true) : attn_plan_make(s[0], s[1], N, D, C, true);
                        if (memcmp(&p, &all, sizeof(p)) != 0) bad("the search leaves out a better plan");
                        ++n;
                    }
                }
    // Beams whose candidates share most of their prefixes: the rows of one or two groups out of many still get
    // workgroups for about half of the chip's 256 compute units and more, as their keys allow (33 tiles of them and more here).
    const int shared[][4] = {{1, 32, 350, 1777}, {1, 32, 350, 4096}, {1, 32, 150, 2048}, {2, 32, 250, 3000}, {4, 40, 80, 4096}, {1, 4, 384, 6000}};
    for (auto &s : shared)
        for (int g = 1; g <= 2; ++g) {
            const AttnPlan p = attn_plan_make(s[0], s[1], s[2], 128, s[3]);
            const int wgs = s[0] * s[1] * g * attn_ranges(p.ranges, g), least = s[0] * s[1] * 10 < 120 ? s[0] * s[1] * 10 : 120;
            if (wgs < least) printf("B=%d H=%d N=%d C=%d: %d workgroups for %d groups of packed rows\n", s[0], s[1], s[2], s[3], wgs, g);
        }
    printf("plans %ld\n", n);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    src, exe = str(tmp / "plan.hip"), str(tmp / "plan")
    with open(src, "w") as f:
        f.write(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2403_09919_amd", "csrc"), "-Wno-unused-function", src, "-o", exe],
                   check=True, capture_output=True, text=True)
    return exe


@pytest.fixture(scope="module")
def report(program):
    return subprocess.run([program], check=True, capture_output=True, text=True, timeout=300).stdout.splitlines()


def test_workspace_layout_is_the_same_for_every_context(report):
    """One workspace may serve calls planned for different contexts (rd_tree_attn_bounded): the completion counters have
    to lie at the same place in front of the partial results whatever the plan."""
    assert report[-1].startswith("plans ") and int(report[-1].split()[1]) > 200000
    assert report[:-1] == [], (len(report) - 1, report[:5])


@pytest.mark.parametrize("way,B,H,W,L,D,C", attn_dealing.SHAPES)
def test_shapes_are_dealt_as_named(program, way, B, H, W, L, D, C):
    for ctx in (C, (C + 31) // 32 * 32):                               # dense, and in pages of 32 keys
        out = subprocess.run([program] + [str(x) for x in (B, H, W * L, D, ctx)], check=True, capture_output=True, text=True).stdout
        assert out.strip() == way
