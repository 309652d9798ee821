"""What a graph and its workspace hold in device memory, against what they held
before searches wrote their output in a dense pass; and that pass's arrays, which
lie in the unused parts of other buffers, over all shares of delegates: searches
of both modes and batches in turn on one workspace, against the oracle."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda
from test_gpu_alloc_failure import CountingAllocator

pytestmark = pytest.mark.gpu

CONTROL = 64 << 10   # control blocks: of fixed size


def _graph(kind, n):
    rng = np.random.default_rng(n)
    if kind == "empty":
        return np.zeros(0, np.int32), np.zeros(0, np.int32), 8
    if kind == "star":                 # one delegate, every other vertex beside it
        v = np.arange(1, n, dtype=np.int32)
        return np.zeros_like(v), v, 4
    if kind == "all":                  # delegates only
        return (rng.integers(0, n, 12 * n, dtype=np.int32),
                rng.integers(0, n, 12 * n, dtype=np.int32), 2)
    # a share of delegates, each with normal neighbours of its own and others
    d = int(n * float(kind))
    src = rng.integers(0, max(d, 1), 10 * n, dtype=np.int32)
    dst = rng.integers(0, n, 10 * n, dtype=np.int32)
    extra = rng.integers(0, n, 2 * n, dtype=np.int32)
    return np.concatenate([src, extra[:n]]), np.concatenate([dst, extra[n:]]), 24


@pytest.mark.parametrize("kind", ["empty", "star", "0.02", "0.2", "0.4", "0.49", "0.6", "all"])
@pytest.mark.parametrize("n", [1, 33, 5000, 200003])
def test_bytes_and_output_in_shared_buffers(oracle_mod, kind, n):
    if n < 33 and kind != "empty":
        pytest.skip("needs vertices")
    d, torch = lib(), torch_cuda()
    src, dst, TH = _graph(kind, n)
    a = CountingAllocator()
    g = d.Graph(src, dst, n, threshold=TH, allocator=a)
    graph_bytes = sum(a.live.values())
    ws = d.Workspace(g, max_lanes=64)
    ws_bytes = sum(a.live.values()) - graph_bytes
    st = g.stats
    nd, nds, nw, dw = st["d"], st["n_ndsrc"], (n + 31) // 32, (st["d"] + 31) // 32
    # bitmaps, two queues, two delegate lists, top-down list and prefix, candidates
    before = 8 * nw + 12 * dw + 8 * n + 8 * nd + 4 * n + 8 * (n + 1) + 8 * nds
    directories = 16 * nw
    log(f"{kind} n={n}: d={nd} nd sources={nds}, workspace {ws_bytes} bytes, before {before}")
    assert ws_bytes + directories <= before + CONTROL
    O = oracle_mod.Graph(src, dst, n)
    label = O.components()
    depth, parent = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    sources = sorted({0, n // 2, n - 1})
    rows = torch.empty((len(sources), n), dtype=torch.int32, device="cuda")
    want = [O.bfs(s, want_parent=False)[0] for s in sources]
    for s, w in zip(sources, want):
        # level by level (a record per level) and in one launch, in turn
        for mode, cap, forced, par in ((1, 64, 0, True), (0, 64, 0, True), (1, 64, 2, True),
                                       (1, 0, 0, True), (1, 64, 2, False), (1, 64, 1, True)):
            depth.fill_(7)
            parent.fill_(7)
            d.bfs(g, ws, s, depth, parent if par else None,
                  opts=d.run_opts(mode=mode, forced=forced, want_parent=par), want_stats=True,
                  capacity=cap)
            torch.cuda.synchronize()
            got = depth.cpu().numpy()
            np.testing.assert_array_equal(got, w, err_msg=f"{kind} {n} {s} {mode} {cap} {forced}")
            if par:
                assert O.check(s, got, parent.cpu().numpy(), label)[0] == 0
        rows.fill_(7)
        d.msbfs(g, ws, sources, rows)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(rows.cpu().numpy(), np.stack(want))
    ws.destroy()
    g.destroy()
    assert not a.live
