"""The dense output pass of searches that run level by level (a call that asks
for a record per level does at any size): depth and parent arrays that begin at
any int32, vertex counts around the row of a thread and the mask word, all
vertices claimed top-down, bottom-up or both, and depths past 255."""
import numpy as np
import pytest

from gpu_helpers import GpuGraph, lib

pytestmark = pytest.mark.gpu

GUARD = 16


def _edges(inputs_mod, kind, n):
    if kind == "path":
        v = np.arange(n - 1, dtype=np.int32)
        return v, v + 1
    src, dst = inputs_mod.rmat_edges(max(1, (n - 1).bit_length()), edge_factor=4, seed=n)
    return (np.ascontiguousarray(src % n, np.int32), np.ascontiguousarray(dst % n, np.int32))


@pytest.mark.parametrize("kind,n", [("path", 2), ("path", 5), ("path", 600), ("rmat", 31),
                                    ("rmat", 33), ("rmat", 1023), ("rmat", 4098)])
def test_outputs_at_any_offset(inputs_mod, oracle_mod, kind, n):
    src, dst = _edges(inputs_mod, kind, n)
    O = oracle_mod.Graph(src, dst, n)
    label = O.components()
    d = lib()
    s = n // 2
    want, _ = O.bfs(s, want_parent=False)
    for TH in (0, 1, 8, 10**6):
        G = GpuGraph(src, dst, n, threshold=TH)
        torch = G.torch
        for off_d, off_p in ((0, 0), (1, 0), (0, 3), (2, 2), (3, None), (0, None)):
            for forced in (0, 1, 2):
                out = torch.full((2, n + 2 * GUARD), 77, dtype=torch.int32, device="cuda")
                depth = out[0, GUARD + off_d - 4:GUARD + off_d - 4 + n]
                parent = None if off_p is None else out[1, GUARD + off_p - 4:GUARD + off_p - 4 + n]
                o = d.run_opts(want_parent=parent is not None, forced=forced)
                d.bfs(G.g, G.ws, s, depth, parent, opts=o, want_stats=True, capacity=1024)
                torch.cuda.synchronize()
                got = depth.cpu().numpy()
                where = f"TH={TH} offsets {off_d} {off_p} forced={forced}"
                np.testing.assert_array_equal(got, want, err_msg=where)
                if parent is not None:
                    assert O.check(s, got, parent.cpu().numpy(), label)[0] == 0, where
                kept = 2 * GUARD + (n + 2 * GUARD if parent is None else 2 * GUARD)
                written = (out.cpu().numpy() == 77)
                inside = (got == 77).sum()
                if parent is not None:
                    inside += (parent.cpu().numpy() == 77).sum()
                assert written.sum() - inside == kept, where
        G.close()
