"""bench.py's command-line contract that can be checked without a GPU: a run on more than one GPU is
refused with a message (this build is single-GPU), and the script never imports the oracle at
module level (the oracle is test infrastructure; only the CPU-baseline leg may load it)."""
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, cwd=ROOT, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr
    assert r.stdout.strip() == ""                       # no JSON line for a run that did not happen


def test_product_code_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2403_09919_amd")
    for name in os.listdir(pkg):
        if name.endswith(".py"):
            src = open(os.path.join(pkg, name)).read()
            assert not re.search(r"^\s*(import|from)\s+oracle\b", src, flags=re.M), name
    bench = open(os.path.join(ROOT, "bench.py")).read()
    top_level = [l for l in bench.splitlines() if re.match(r"(import|from)\s+oracle\b", l)]
    assert top_level == []                              # only inside cpu_baseline()
    assert re.search(r"def cpu_baseline\(.*?\n(.*\n)*?\s+import oracle", bench)


def test_traffic_is_reported_only_for_the_kernel_it_was_measured_on(tmp_path):
    """The counter summary names the sources it was measured on; with other sources its figures are not reported."""
    import bench
    src = tmp_path / "kernel.h"
    src.write_text("int a = 1; // one\n")
    measured = bench.attention_digest([src])
    table = tmp_path / "table.md"
    table.write_text("sources: %s\n| 2 | 1.0 | 2.0 | 1 | 1 | 4096 |\n" % measured)
    assert bench.read_traffic_table(table, measured) == {2: 4096}
    src.write_text("int a =\n  1; // another comment\n")
    assert bench.read_traffic_table(table, bench.attention_digest([src])) == {2: 4096}
    src.write_text("int a = 2; // one\n")
    assert bench.read_traffic_table(table, bench.attention_digest([src])) == {}
    table.write_text("| 2 | 1.0 | 2.0 | 1 | 1 | 4096 |\n")
    assert bench.read_traffic_table(table, measured) == {}


def test_traffic_depends_on_every_file_of_the_attention_kernel():
    """What the 16-bit kernel and its entry points are made of, header by header, is what the counter summary is tied to."""
    import bench
    csrc = os.path.join(ROOT, "paper_2403_09919_amd", "csrc")
    todo, files = ["rd_tree_attn.hip", "rd_tree_attn_bf16.hip"], set()
    while todo:
        name = todo.pop()
        if name in files or not os.path.exists(os.path.join(csrc, name)):
            continue
        files.add(name)
        todo += re.findall(r'#include "([^"]+)"', open(os.path.join(csrc, name)).read())
    assert sorted(os.path.basename(p) for p in bench.ATTENTION_SOURCES) == sorted(files)
