"""The rule that chooses a one-launch search's grid (bfs.hip), on the host: by
vertices where edges are few a vertex, wider with the edges that the search
reads, and never narrower for more of them. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
DO, TD, PLAIN = (1, 0, 0.02), (1, 1, 0.02), (0, 0, 0.02)
NEVER_BACK = (1, 0, 1e9)


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    tmp = tmp_path_factory.mktemp("shape")
    text = open(os.path.join(ROOT, "paper_1803_03922_amd", "csrc", "bfs.hip")).read()
    parts = [re.search(r"struct OneLaunch \{.*?\n\};\n", text, re.S).group(0)]
    parts += re.findall(r"^OneLaunch \w+_shape\(.*?\n\}\n", text, re.S | re.M)
    (tmp / "shape.inc").write_text("\n".join(parts))
    exe = str(tmp / "shape")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(tmp), "-I", os.path.join(ROOT, "include"),
                    "-o", exe, os.path.join(HERE, "emulation", "shape.cpp")], check=True)

    def run(rows):
        text = "\n".join(" ".join(str(x) for x in (*how, n, m, mx)) for how, n, m, mx in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


def test_sparse_graphs_by_vertices(shapes):
    """16 and 24 pairs a vertex: the lines lie where they are by vertices alone."""
    want = {PLAIN: [(1 << 13, (32, 256)), (1 << 15, (64, 256)), (3 << 15, (64, 512)),
                    (3 << 17, (128, 512)), (3 << 19, (256, 512)), (3 << 20, (256, 1024)),
                    (1 << 27, (0, 0))],
            DO: [(1 << 14, (32, 256)), (3 << 16, (64, 512)), (3 << 20, (128, 1024)),
                 (3 << 22, (256, 1024)), (1 << 27, (0, 0))]}
    for how, lines in want.items():
        first = 1
        for last, shape in lines:
            for degree, mx in ((32, 40), (47, 10**6), (2, 3)):
                got = shapes([(how, n, degree * n, mx) for n in (first, last)])
                assert got == [shape, shape], (how, first, last, degree)
            first = last + 1


def test_dense_graphs(shapes):
    rows = [(PLAIN, 1 << 13, 33_000_000, 8000), (PLAIN, 1 << 14, 106_000_000, 6600),
            (PLAIN, 1 << 18, 134_000_000, 700), (TD, 1 << 14, 23_000_000, 16000),
            (NEVER_BACK, 1 << 14, 23_000_000, 16000), (DO, 1 << 14, 23_000_000, 16000),
            (DO, 1 << 14, 32_000_000, 2200), (DO, 1 << 20, 134_000_000, 180),
            (DO, 1 << 12, 15_000_000, 3700)]
    assert shapes(rows) == [(256, 512), (256, 1024), (256, 512), (128, 512), (128, 512), (32, 256),
                            (128, 1024), (256, 1024), (32, 256)]


@pytest.mark.parametrize("how", [DO, TD, PLAIN, NEVER_BACK])
def test_never_narrower_for_more(shapes, how):
    """More edges on the same vertices never make the grid narrower (the widest is
    level by level), for a uniform graph and one with hubs."""
    def width(s):
        return s[0] * s[1] or 1 << 30
    ns = [int(2 ** (i / 4)) for i in range(8, 104)]
    for hub in (False, True):
        table = {}
        for k in range(0, 16):
            got = shapes([(how, n, n << k, n - 1 if hub else (n << k) // n) for n in ns])
            table[k] = [width(s) for s in got]
        for k in range(1, 16):
            # (up to half of all the edges there can be)
            assert all(a <= b for n, a, b in zip(ns, table[k - 1], table[k]) if 2 << k <= n), (hub, k)
