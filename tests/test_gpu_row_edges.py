"""Row lengths where the builder, PageRank and multi-source BFS change kernels
(rows up to 64 and up to 8192 entries, a delegate row read by several blocks
past 4096 entries, a hub row set aside past 1088), one entry either side, and
edge lists around the tiles of the packing and sorting passes, against the
oracle. PageRank's tolerance is test_gpu_pagerank's: FP64 sums in another
order, 1e-10 relative, 1e-18 absolute."""
import numpy as np
import pytest

import test_gpu_bfs
import test_gpu_msbfs
from gpu_helpers import lib, torch_cuda

pytestmark = pytest.mark.gpu

LENGTHS = (63, 64, 65, 511, 512, 513, 1024, 1088, 1089, 1152, 4095, 4096, 4097, 8191, 8192, 8193,
           16000)


def _stars(n=20011):
    """Vertices 0.. of the lengths above, each with that many distinct leaves, and
    a sparse ring through all vertices."""
    rng = np.random.default_rng(5)
    src, dst = [], []
    hubs = len(LENGTHS)
    for h, k in enumerate(LENGTHS):
        leaf = rng.choice(np.arange(hubs, n), k, replace=False)
        src.append(np.full(k, h))
        dst.append(leaf)
    ring = np.arange(hubs, n - 1)[::3]
    src.append(ring)
    dst.append(ring + 1)
    return n, np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)


@pytest.mark.parametrize("TH", [0, 2, 64, 512, 4096, 10**6])
def test_layout_at_row_lengths(inputs_mod, oracle_mod, monkeypatch, TH):
    n, src, dst = _stars()
    O = oracle_mod.Graph(src, dst, n)
    monkeypatch.setattr(test_gpu_bfs, "_rmat", lambda *a: (n, src, dst, O))
    test_gpu_bfs.test_builder_layout_matches_oracle_split(inputs_mod, oracle_mod, 0, TH)


@pytest.mark.parametrize("edges", [1, 63, 64, 65, 4095, 4096, 4097, 8191, 8193, 16385])
def test_layout_at_tile_edges(inputs_mod, oracle_mod, monkeypatch, edges):
    n = 1031
    rng = np.random.default_rng(edges)
    src = rng.integers(0, n, edges, dtype=np.int32)
    dst = rng.integers(0, n, edges, dtype=np.int32)
    O = oracle_mod.Graph(src, dst, n)
    monkeypatch.setattr(test_gpu_bfs, "_rmat", lambda *a: (n, src, dst, O))
    test_gpu_bfs.test_builder_layout_matches_oracle_split(inputs_mod, oracle_mod, 0, 8)


@pytest.mark.parametrize("TH", [2, 600])
def test_pagerank_and_batches_at_row_lengths(oracle_mod, TH):
    n, src, dst = _stars()
    d = lib()
    torch = torch_cuda()
    O = oracle_mod.Graph(src, dst, n)
    g = d.Graph(src, dst, n, threshold=TH)
    rank = torch.empty(n, dtype=torch.float64, device="cuda")
    for iters in (0, 1, 12):
        assert d.pagerank(g, rank, iterations=iters)[0] == iters
        torch.cuda.synchronize()
        np.testing.assert_allclose(rank.cpu().numpy(), O.pagerank(0.85, iters), rtol=1e-10,
                                   atol=1e-18)
    sources = list(range(len(LENGTHS))) + list(range(100, n, 401))
    want = [O.bfs(s, want_parent=False)[0] for s in sources]
    ws = d.Workspace(g, max_lanes=64)
    depth = torch.empty((len(sources), n), dtype=torch.int32, device="cuda")
    for permille in (0, 1, 50, 1000):
        depth.fill_(7)
        o = test_gpu_msbfs._opts(permille=permille, lanes=64)
        d.msbfs(g, ws, sources, depth, o)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(depth.cpu().numpy(), np.stack(want))
    ws.destroy()
    g.destroy()
