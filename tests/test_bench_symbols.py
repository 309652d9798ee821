"""The kernel names by which the bench looks up measured traffic are those of
kernels in the source, one for every visit that a search reports. CPU only."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_kernel_symbols_are_kernels():
    from paper_1803_03922_amd import dsbfs
    assert set(bench.KERNEL_SYMBOL) == set(dsbfs.KERNEL_NAMES)
    text = open(os.path.join(ROOT, "paper_1803_03922_amd", "csrc", "bfs.hip")).read()
    bits = dict(re.findall(r"(k\w+) = (\d+)", re.search(r"enum \{ (kDeleg = 1.*?) \};", text).group(1)))
    launched = {"k_init", "k_bu_nn", "k_plain_expand"}
    for name, parts in re.findall(r"\((k_\w+)<([\w| ]+)>\)", text):
        launched.add(f"{name}<{sum(int(bits[p.strip()]) for p in parts.split('|'))}>")
    assert set(bench.KERNEL_SYMBOL.values()) <= launched
