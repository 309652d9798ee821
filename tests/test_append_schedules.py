"""The append step of the bottom-up normal visit under wave schedules that the
hardware allows but seldom takes: the step's own lines (bfs.hip) and the
append buffers (internal.hpp) run on the CPU as one block whose lanes are
fibers, with single waves let ahead of the others between two barriers. Every
wave must pass the same barriers, and both lists hold what was pushed. CPU
only."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1803_03922_amd", "csrc")


def _text(name):
    return open(os.path.join(CSRC, name)).read()


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    tmp = tmp_path_factory.mktemp("append")
    text = _text("internal.hpp")
    append = re.search(r"struct BlockAppend \{.*?\n\};\n", text, re.S).group(0)
    append += "\n".join(re.findall(r"__device__ inline void flush_pair\w*\(.*?\n\}\n", text, re.S))
    step = re.search(r"void bu_normal\(.*?\n(    qa\.push\(won, v\);.*?)\n  \}\n  flush_pair\(qa, ca\);",
                     _text("bfs.hip"), re.S).group(1)
    (tmp / "append.inc").write_text(append)
    (tmp / "step.inc").write_text(step)
    exe = str(tmp / "append_step")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", str(tmp), "-o", exe,
                    os.path.join(HERE, "emulation", "append_step.cpp")], check=True)
    return exe


# waves and capacity as the kernels have them, and small blocks; densities from
# buffers that a flush just misses to buffers that overflow
@pytest.mark.parametrize("waves,cap", [(2, 192), (4, 1408), (16, 3072)])
@pytest.mark.parametrize("density", [0.05, 0.3, 0.7, 1.0])
def test_append_step_under_schedules(driver, waves, cap, density):
    r = subprocess.run([driver, str(waves), str(cap), "24", str(density)], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "append step ok" in r.stdout
