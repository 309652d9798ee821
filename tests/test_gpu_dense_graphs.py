"""Searches in one launch of graphs with many edges a vertex, whose grids follow
the edges: uniform graphs and RMAT graphs, both modes, top-down and bottom-up
schedules, against the oracle."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,pairs", [
    ("er", 1030, 1 << 19), ("er", 1030, (1 << 20) + 9), ("er", 5000, 3 << 20), ("er", 9000, 8 << 20),
    ("rmat", 1 << 12, 2 << 20), ("rmat", 1 << 14, 8 << 20), ("er", 140000, 8 << 20)])
def test_dense_graphs(inputs_mod, oracle_mod, kind, n, pairs):
    d, torch = lib(), torch_cuda()
    rng = np.random.default_rng(pairs)
    if kind == "rmat":
        src, dst = inputs_mod.rmat_edges((n - 1).bit_length(), edge_factor=pairs // n, seed=3)
    else:
        src, dst = (rng.integers(0, n, pairs, dtype=np.int32) for _ in range(2))
    O = oracle_mod.Graph(src, dst, n)
    label = O.components()
    s = int(inputs_mod.pick_sources(src, dst, n, 1, seed=6)[0])
    want, _ = O.bfs(s, want_parent=False)
    for TH in (32, 10**6):
        g = d.Graph(src, dst, n, threshold=TH)
        ws = d.Workspace(g)
        depth, parent = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
        for kw in ({}, {"mode": 0}, {"forced": 1}, {"forced": 2}, {"factor0": (1e9, 1e9, 1e9)},
                   {"nn_do": True, "factor_nn": (1e-6, 0.0)}):
            depth.fill_(7)
            parent.fill_(7)
            st = d.bfs(g, ws, s, depth, parent, opts=d.run_opts(**kw), want_stats=True, capacity=0)
            torch.cuda.synchronize()
            got = depth.cpu().numpy()
            np.testing.assert_array_equal(got, want, err_msg=f"TH={TH} {kw}")
            assert O.check(s, got, parent.cpu().numpy(), label)[0] == 0, (TH, kw)
            assert st["reached"] == int((want >= 0).sum())
        log(f"dense {kind} n={n} m={g.stats['m_dir']} TH={TH} ok")
        ws.destroy()
        g.destroy()
