"""Searches of more levels than one launch runs (252): the launches that go on
where the one before ended, on paths around multiples of that, and with a uniform
core at the far end, whose heavy levels come in a later launch; all modes, the
allocation-free call, statistics, and a launch that gives up. And a batch beside
a search of many launches. Against closed forms and the oracle."""
import threading
import time

import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda
from test_gpu_one_launch_fallback import _bound

pytestmark = pytest.mark.gpu

KWS = ({}, {"mode": 0}, {"forced": 1}, {"forced": 2}, {"nn_do": True, "factor_nn": (1e-6, 0.0)},
       {"want_parent": False}, {"mode": 0, "want_parent": False})


def _search_all(d, torch, g, ws, n, s, want, check, kws=KWS):
    depth, parent = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    for kw in kws:
        par = kw.get("want_parent", True)
        o = d.run_opts(**kw)
        for call in ("bfs", "noalloc"):
            depth.fill_(7)
            parent.fill_(7)
            p = parent if par else None
            if call == "bfs":
                st = d.bfs(g, ws, s, depth, p, opts=o, want_stats=True, capacity=0)
                reached = want >= 0
                assert st["reached"] == int(reached.sum()), (kw, call)
                assert st["num_levels"] == int(want.max()) + 1, (kw, call)
            else:
                d.bfs_noalloc(g, s, depth, p, opts=o)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(depth.cpu().numpy(), want, err_msg=f"{kw} {call}")
            if par:
                check(depth.cpu().numpy(), parent.cpu().numpy(), (kw, call))


@pytest.mark.parametrize("n", [251, 252, 253, 254, 255, 503, 505, 1300])
def test_paths_around_a_launch(oracle_mod, n):
    d, torch = lib(), torch_cuda()
    v = np.arange(n - 1, dtype=np.int32)
    # TH 1: the inner vertices are delegates; TH 2: none is
    for TH in (1, 2):
        g = d.Graph(v, v + 1, n, threshold=TH)
        ws = d.Workspace(g)

        def check(depth, parent, what):
            np.testing.assert_array_equal(parent, np.maximum(np.arange(n) - 1, 0), err_msg=str(what))
        _search_all(d, torch, g, ws, n, 0, np.arange(n), check)
        ws.destroy()
        g.destroy()


@pytest.mark.parametrize("tail", [100, 250, 251, 252, 600])
@pytest.mark.parametrize("TH", [12, 10**6])
def test_heavy_levels_in_a_later_launch(oracle_mod, tail, TH):
    d, torch = lib(), torch_cuda()
    core = 600000
    n = core + tail
    rng = np.random.default_rng(tail)
    src, dst = (rng.integers(0, core, 8 * core, dtype=np.int32) for _ in range(2))
    v = np.arange(core, n - 1, dtype=np.int32)
    src = np.concatenate([src, v, [core]]).astype(np.int32)
    dst = np.concatenate([dst, v + 1, [5]]).astype(np.int32)
    O = oracle_mod.Graph(src, dst, n)
    want, _ = O.bfs(n - 1, want_parent=False)
    assert want.max() > tail
    label = O.components()
    g = d.Graph(src, dst, n, threshold=TH)
    ws = d.Workspace(g)

    def check(depth, parent, what):
        assert O.check(n - 1, depth, parent, label)[0] == 0, what
    _search_all(d, torch, g, ws, n, n - 1, want, check, KWS[:2] + KWS[5:])
    # a launch that gives up, and the search again level by level
    depth = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    _bound(d, ws, -1)
    d.bfs(g, ws, n - 1, depth, None, opts=d.run_opts(want_parent=False))
    assert _bound(d, ws, 0) == 16
    np.testing.assert_array_equal(depth.cpu().numpy(), want)
    ws.destroy()
    g.destroy()


def test_batch_beside_a_search_of_many_launches(inputs_mod, oracle_mod):
    d, torch = lib(), torch_cuda()
    n = 1 << 14
    src, dst = inputs_mod.rmat_edges(14)
    O = oracle_mod.Graph(src, dst, n)
    sources = inputs_mod.pick_sources(src, dst, n, 6, seed=11).tolist()
    want = np.stack([O.bfs(s, want_parent=False)[0] for s in sources])
    g = d.Graph(src, dst, n, threshold=32)
    wb = d.Workspace(g, max_lanes=64)
    rows = torch.empty((len(sources), n), dtype=torch.int32, device="cuda")
    long = 120000
    v = np.arange(long - 1, dtype=np.int32)
    path = d.Graph(v, v + 1, long, threshold=32, keep_plain_csr=False)
    ws = d.Workspace(path)
    depth = torch.empty(long, dtype=torch.int32, device="cuda")
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    d.msbfs(g, wb, sources, rows, stream=two.cuda_stream)
    ended, errors = threading.Event(), []

    def search():
        try:
            d.bfs(path, ws, 0, depth, None, opts=d.run_opts(want_parent=False),
                  stream=one.cuda_stream)
        except Exception as e:
            errors.append(e)
        ended.set()

    t = threading.Thread(target=search)
    t.start()
    time.sleep(0.05)
    took = []
    for _ in range(4):
        rows.fill_(7)
        torch.cuda.current_stream().synchronize()
        t0 = time.monotonic()
        d.msbfs(g, wb, sources, rows, stream=two.cuda_stream)
        took.append(round((time.monotonic() - t0) * 1e3, 2))
        assert np.array_equal(rows.cpu().numpy(), want)
    before = not ended.is_set()
    t.join()
    log(f"batches beside a search of {long} levels: {took} ms")
    assert not errors, errors
    np.testing.assert_array_equal(depth.cpu().numpy(), np.arange(long))
    assert before, f"the batches returned only after the search: {took} ms"
    path.destroy()
    g.destroy()
