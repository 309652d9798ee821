"""Searches in one launch at the vertex counts where the grid changes, the last
of one shape and the first of the next: every option up to 3 * 2^17 vertices,
and beyond it, with a sparse graph, the default search and the plain one, up to
where searches go level by level. Against the oracle."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda

pytestmark = pytest.mark.gpu

ALL = ({}, {"mode": 0}, {"forced": 1}, {"forced": 2}, {"want_parent": False},
       {"nn_do": True, "factor_nn": (1e-6, 0.0)}, {"factor1": (1.0, 1.0, 1.0)})
FEW = ({}, {"mode": 0, "want_parent": False})


def _check(d, torch, O, g, n, sources, kws, label):
    ws = d.Workspace(g)
    depth, parent = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    for s in sources:
        want, _ = O.bfs(s, want_parent=False)
        for kw in kws:
            par = kw.get("want_parent", True)
            depth.fill_(7)
            parent.fill_(7)
            st = d.bfs(g, ws, s, depth, parent if par else None, opts=d.run_opts(**kw),
                       want_stats=True, capacity=0)
            torch.cuda.synchronize()
            got = depth.cpu().numpy()
            np.testing.assert_array_equal(got, want, err_msg=f"n={n} {s} {kw}")
            assert st["reached"] == int((want >= 0).sum())
            if par:
                assert O.check(s, got, parent.cpu().numpy(), label)[0] == 0, (n, s, kw)
    ws.destroy()


@pytest.mark.parametrize("edge", [1 << 13, 1 << 14, 1 << 15, 3 << 15, 3 << 16, 3 << 17])
def test_both_sides_of_small_edges(inputs_mod, oracle_mod, edge):
    d, torch = lib(), torch_cuda()
    for n in (edge, edge + 1):
        src, dst = inputs_mod.rmat_edges((n - 1).bit_length(), edge_factor=6, seed=n)
        src, dst = (np.ascontiguousarray(x % n, np.int32) for x in (src, dst))
        O = oracle_mod.Graph(src, dst, n)
        sources = inputs_mod.pick_sources(src, dst, n, 2, seed=1).tolist()
        label = O.components()
        for TH in (16, 10**6):
            g = d.Graph(src, dst, n, threshold=TH)
            _check(d, torch, O, g, n, sources, ALL, label)
            g.destroy()
    log(f"edge {edge} ok")


@pytest.mark.parametrize("edge", [3 << 19, 3 << 20, 3 << 22])
def test_both_sides_of_large_edges(oracle_mod, edge):
    d, torch = lib(), torch_cuda()
    rng = np.random.default_rng(edge)
    for n in (edge, edge + 1):
        # two uniform pairs a vertex, and hubs
        src = rng.integers(0, n, 2 * n, dtype=np.int32)
        dst = rng.integers(0, n, 2 * n, dtype=np.int32)
        src[:n // 8] = rng.integers(0, 500, n // 8)
        O = oracle_mod.Graph(src, dst, n)
        label = O.components()
        g = d.Graph(src, dst, n, threshold=32)
        _check(d, torch, O, g, n, [int(src[-1])], FEW, label)
        g.destroy()
        log(f"edge {edge}, n={n} ok")
