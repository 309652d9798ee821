"""Single-source searches in one launch against the level-by-level driver and
the oracle. A call that asks for a record per level runs level by level, one
that does not runs in one launch where the graph is small enough; both must
give the oracle's depths and valid parents, and the same statistics. Sizes sit
at the edges: of a mask word, of the grid shapes' ranges, of the forward list's
segments and of a wave's 64 rows."""
import threading

import numpy as np
import pytest

from gpu_helpers import GpuGraph, lib, log, torch_cuda

pytestmark = pytest.mark.gpu


def _graph(inputs_mod, kind, n):
    rng = np.random.default_rng(n)
    if kind == "rmat":
        levels = max(1, (n - 1).bit_length())
        src, dst = inputs_mod.rmat_edges(levels, edge_factor=8, seed=n)
        return src % n, dst % n
    if kind == "er":
        return (rng.integers(0, n, 6 * n, dtype=np.int32),
                rng.integers(0, n, 6 * n, dtype=np.int32))
    if kind == "path":
        v = np.arange(n - 1, dtype=np.int32)
        return v, v + 1
    # two hubs sharing every leaf: rows much longer than a wave's steps
    v = np.arange(2, n, dtype=np.int32)
    return (np.concatenate([np.zeros_like(v), np.ones_like(v)]), np.concatenate([v, v]))


@pytest.mark.parametrize("kind,n", [
    ("path", 2), ("path", 33), ("path", 700), ("hubs", 3), ("hubs", 66), ("hubs", 70000),
    ("rmat", 31), ("rmat", 65), ("rmat", 1025), ("rmat", 32768), ("rmat", 32769),
    ("rmat", 131073), ("er", 64), ("er", 4097), ("er", 40000)])
def test_one_launch_equals_levels_and_oracle(inputs_mod, oracle_mod, kind, n):
    src, dst = _graph(inputs_mod, kind, n)
    src, dst = np.ascontiguousarray(src, np.int32), np.ascontiguousarray(dst, np.int32)
    d = lib()
    O = oracle_mod.Graph(src, dst, n)
    label = O.components()
    for TH in (0, 4, 32, 10**6):
        G = GpuGraph(src, dst, n, threshold=TH)
        torch = G.torch
        for s in sorted({0, n // 2, n - 1}):
            want, _ = O.bfs(s, want_parent=False)
            for kw in ({}, {"mode": 0}, {"forced": 1}, {"forced": 2}, {"forced": 3, "seed": 5},
                       {"nn_do": True, "factor_nn": (1e-6, 0.0)}, {"factor1": (1.0, 1.0, 1.0)}):
                depth, parent, st = G.bfs(s, want_stats=True, **kw)      # level by level
                np.testing.assert_array_equal(depth, want, err_msg=f"levels TH={TH} {s} {kw}")
                assert O.check(s, depth, parent, label)[0] == 0
                opts = dict(kw)
                opts["forced_seed"] = opts.pop("seed", 0)
                o = d.run_opts(**opts)
                G.depth.fill_(7)
                G.parent.fill_(7)
                one = d.bfs(G.g, G.ws, s, G.depth, G.parent, opts=o, want_stats=True, capacity=0)
                torch.cuda.synchronize()
                depth, parent = G.depth[:n].cpu().numpy(), G.parent[:n].cpu().numpy()
                np.testing.assert_array_equal(depth, want, err_msg=f"one launch TH={TH} {s} {kw}")
                assert O.check(s, depth, parent, label)[0] == 0
                for k in ("num_levels", "reached", "edges_cc"):
                    assert one[k] == st[k], (k, TH, s, kw)
        G.close()
    log(f"one launch {kind} n={n} ok")


def test_concurrent_searches_and_batches(inputs_mod, oracle_mod):
    """Searches in one launch from several threads, each with its workspace and
    stream, beside multi-source batches: every grid that waits for its own
    blocks completes, and every row is the oracle's."""
    d = lib()
    torch = torch_cuda()
    scale = 15
    n = 1 << scale
    src, dst = inputs_mod.rmat_edges(scale)
    O = oracle_mod.Graph(src, dst, n)
    g = d.Graph(src, dst, n, threshold=16)
    sources = inputs_mod.pick_sources(src, dst, n, 16, seed=5).tolist()
    want = {s: O.bfs(s, want_parent=False)[0] for s in sources}
    bad, errors = [], []

    def searches(k):
        try:
            stream = torch.cuda.Stream()
            ws = d.Workspace(g)
            depth = torch.empty(n, dtype=torch.int32, device="cuda")
            for i in range(24):
                s = sources[(i + 3 * k) % len(sources)]
                d.bfs(g, ws, s, depth, None, opts=d.run_opts(want_parent=False, mode=i % 2),
                      stream=stream.cuda_stream)
                stream.synchronize()
                if not np.array_equal(depth.cpu().numpy(), want[s]):
                    bad.append((k, i, s))
        except Exception as e:
            errors.append(e)

    def batches():
        try:
            stream = torch.cuda.Stream()
            ws = d.Workspace(g, max_lanes=64)
            depth = torch.empty((len(sources), n), dtype=torch.int32, device="cuda")
            for i in range(6):
                d.msbfs(g, ws, sources, depth, stream=stream.cuda_stream)
                got = depth.cpu().numpy()
                for j, s in enumerate(sources):
                    if not np.array_equal(got[j], want[s]):
                        bad.append(("batch", i, s))
        except Exception as e:
            errors.append(e)

    threads = [threading.Thread(target=searches, args=(k,)) for k in range(4)]
    threads.append(threading.Thread(target=batches))
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert not bad, bad
    g.destroy()
