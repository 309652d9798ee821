"""A first batch on a workspace that fails at any of its allocations, then a
batch on another stream: what the first left (the hub list, the columns with hub
slots) is complete for the second, whose rows are the oracle's."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda
from test_gpu_alloc_failure import CountingAllocator

pytestmark = pytest.mark.gpu


def test_batch_after_a_failed_first_one(inputs_mod, oracle_mod):
    d, torch = lib(), torch_cuda()
    n = 1 << 15
    src, dst = inputs_mod.rmat_edges(15, edge_factor=32)
    O = oracle_mod.Graph(src, dst, n)
    sources = inputs_mod.pick_sources(src, dst, n, 5, seed=4).tolist()
    want = np.stack([O.bfs(s, want_parent=False)[0] for s in sources])
    a = CountingAllocator()
    g = d.Graph(src, dst, n, threshold=32, allocator=a)
    rows = torch.empty((len(sources), n), dtype=torch.int32, device="cuda")
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    failed = 0
    while True:
        ws = d.Workspace(g, max_lanes=64)
        rows.fill_(7)
        torch.cuda.synchronize()
        a.fail_at = a.requests + failed
        try:
            d.msbfs(g, ws, sources, rows, stream=one.cuda_stream)
            done = True
        except d.DsbfsError as e:
            assert e.status == d.ERR_OUT_OF_MEMORY
            done = False
        a.fail_at = None
        d.msbfs(g, ws, sources, rows, stream=two.cuda_stream)
        np.testing.assert_array_equal(rows.cpu().numpy(), want, err_msg=f"request {failed}")
        ws.destroy()
        if done:
            break
        failed += 1
    log(f"batches after failures at {failed} requests ok")
    assert failed >= 8
    g.destroy()
    assert not a.live
