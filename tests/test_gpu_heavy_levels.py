"""Levels whose nn visit scatters and settles (long normal rows, a frontier with
many edges to unvisited vertices, graphs of some 300k vertices and more) against
the oracle and the level-by-level driver: vertex counts around a wave's group of
64 and a mask word, with and without parents, delegates beside normals or none,
and both directions forced."""
import numpy as np
import pytest

from gpu_helpers import GpuGraph, lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,degree,thresholds", [
    (300031, 16, (16, 10**6)), (327680, 8, (10**6,)), (327681, 8, (7,)),
    (400063, 24, (24, 10**6)), (1 << 20, 16, (10**6,))])
def test_scatter_levels_equal_levels_and_oracle(inputs_mod, oracle_mod, n, degree, thresholds):
    rng = np.random.default_rng(n)
    m = n * degree // 2
    src = rng.integers(0, n, m, dtype=np.int32)
    dst = rng.integers(0, n, m, dtype=np.int32)
    O = oracle_mod.Graph(src, dst, n)
    label = O.components()
    d = lib()
    s = int(src[0])
    want, _ = O.bfs(s, want_parent=False)
    for TH in thresholds:
        G = GpuGraph(src, dst, n, threshold=TH)
        for kw in ({}, {"forced": 1}, {"forced": 2}):
            depth, parent, st = G.bfs(s, want_stats=True, **kw)     # level by level
            np.testing.assert_array_equal(depth, want)
            for parents in (True, False):
                G.depth.fill_(7)
                G.parent.fill_(7)
                o = d.run_opts(want_parent=parents, **kw)
                one = d.bfs(G.g, G.ws, s, G.depth, G.parent if parents else None, opts=o,
                            want_stats=True, capacity=0)
                G.torch.cuda.synchronize()
                where = f"n={n} TH={TH} {kw} parents={parents}"
                got = G.depth[:n].cpu().numpy()
                np.testing.assert_array_equal(got, want, err_msg=where)
                if parents:
                    assert O.check(s, got, G.parent[:n].cpu().numpy(), label)[0] == 0, where
                for k in ("num_levels", "reached", "edges_cc"):
                    assert one[k] == st[k], (k, where)
        G.close()
