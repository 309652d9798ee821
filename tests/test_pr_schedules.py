"""The block sums of PageRank's delegate pull under wave schedules that the
hardware allows but seldom takes: the kernel's own lines (pagerank.hip) run on
the CPU as one block whose lanes are fibers, with single waves let ahead of the
others between two barriers. Whole numbers, so sums are exact. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1803_03922_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_block_rows_then_block_sum_under_schedules(tmp_path):
    text = open(os.path.join(CSRC, "pagerank.hip")).read()
    sums = "\n".join(re.search(rf"__device__ __forceinline__ \w+ {f}\(.*?\n\}}\n", text, re.S).group(0)
                     for f in ("wave_sum_f64", "block_add_f64"))
    kernel = text[text.index("k_pr_deleg(PrStep a"):]
    rows = re.search(r"kDW \* kPrUnroll \* kWave\)\);\n(.*?\n  \})\n  const int64_t nw", kernel,
                     re.S).group(1)
    (tmp_path / "sum.inc").write_text(sums)
    (tmp_path / "rows.inc").write_text(rows)
    exe = str(tmp_path / "pr_lead_rows")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", str(tmp_path), "-o", exe,
                    os.path.join(HERE, "emulation", "pr_lead_rows.cpp")], check=True)
    for count in (1, 2, 5):
        r = subprocess.run([exe, str(count)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, f"{count} rows: {r.stdout}{r.stderr}"
        assert "rows ok" in r.stdout
