"""The gate that hands out compute units to grids that wait for their own
blocks: its code (bfs.hip) on the host, with devices of 256, 32 and 80 units.
CPU only."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1803_03922_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_gate(tmp_path):
    text = open(os.path.join(CSRC, "bfs.hip")).read()
    gate = re.search(r"namespace \{\nstruct ResidentGate \{.*?ResidentLease::~ResidentLease\(\) \{.*?\n\}\n",
                     text, re.S).group(0)
    (tmp_path / "gate.inc").write_text(gate)
    exe = str(tmp_path / "gate")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I",
                    str(tmp_path), "-o", exe, os.path.join(HERE, "emulation", "gate.cpp")],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "gate ok" in r.stdout
