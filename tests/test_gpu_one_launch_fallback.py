"""Searches in one launch whose blocks cannot all run: the launch gives up, the
search runs level by level with the same results, and the workspace's next
searches do not try again at once. The bound of a wait is set from the host
(every kernel ends normally), or another stream's kernel holds a compute unit."""
import ctypes
import time

import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda
from test_gpu_gate import _beside, _sleep

pytestmark = pytest.mark.gpu


def _bound(d, ws, ticks):
    f = ctypes.CDLL(d.LIB_PATH).dsbfs_test_barrier_bound
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int64], ctypes.c_int32
    return f(ws.h, ticks)


@pytest.mark.parametrize("kw", [{}, {"mode": 0}, {"nn_do": True, "factor_nn": (1e-6, 0.0)}],
                         ids=["do", "plain", "nn_do"])
@pytest.mark.parametrize("kind,n", [("rmat", 1000), ("rmat", 70000), ("er", 300001)])
def test_gives_up_and_goes_level_by_level(inputs_mod, oracle_mod, kind, n, kw):
    d, torch = lib(), torch_cuda()
    rng = np.random.default_rng(n)
    if kind == "rmat":
        src, dst = inputs_mod.rmat_edges((n - 1).bit_length(), edge_factor=8, seed=n)
        src, dst = src % n, dst % n
    else:
        src, dst = (rng.integers(0, n, 8 * n, dtype=np.int32) for _ in range(2))
    src, dst = np.ascontiguousarray(src, np.int32), np.ascontiguousarray(dst, np.int32)
    O = oracle_mod.Graph(src, dst, n)
    label = O.components()
    g = d.Graph(src, dst, n, threshold=16)
    ws = d.Workspace(g)
    depth, parent = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    s = int(inputs_mod.pick_sources(src, dst, n, 1, seed=2)[0])
    want, _ = O.bfs(s, want_parent=False)

    def search():
        depth.fill_(7)
        parent.fill_(7)
        st = d.bfs(g, ws, s, depth, parent, opts=d.run_opts(**kw), want_stats=True, capacity=0)
        torch.cuda.synchronize()
        got = depth.cpu().numpy()
        np.testing.assert_array_equal(got, want)
        assert O.check(s, got, parent.cpu().numpy(), label)[0] == 0
        return st["num_levels"], st["reached"], st["edges_cc"]

    right = search()                      # in one launch
    assert _bound(d, ws, -1) == 0
    assert search() == right              # gives up, then level by level
    for left in range(16, 0, -1):         # the next ones do not try
        assert _bound(d, ws, -1) == left
        assert search() == right
    assert _bound(d, ws, -1) == 0
    assert search() == right              # tries and gives up again
    assert _bound(d, ws, 0) == 64
    for _ in range(64):
        d.bfs(g, ws, s, depth, parent, opts=d.run_opts(**kw))
    assert _bound(d, ws, 0) == 0
    assert search() == right              # in one launch again
    assert _bound(d, ws, -1) == 0
    assert search() == right
    assert _bound(d, ws, 0) == 16         # a success had set the count back
    ws.destroy()
    g.destroy()


def test_search_beside_another_streams_kernel(oracle_mod):
    """A graph whose search takes a block of 1024 threads on every compute unit,
    beside a kernel of one wave that runs for longer than all the searches."""
    d, torch = lib(), torch_cuda()
    n = (3 << 20) + 12345
    rng = np.random.default_rng(4)
    src, dst = (rng.integers(0, n, 3 * n, dtype=np.int32) for _ in range(2))
    want, _ = oracle_mod.Graph(src, dst, n).bfs(5, want_parent=False)
    g = d.Graph(src, dst, n, threshold=32, keep_plain_csr=False)
    ws = d.Workspace(g)
    depth = torch.empty(n, dtype=torch.int32, device="cuda")
    one = torch.cuda.Stream()
    o = d.run_opts(want_parent=False)
    d.bfs(g, ws, 5, depth, None, opts=o, stream=one.cuda_stream)

    class T:
        pass
    T.torch, T.probe = torch, torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    ended = _sleep(T, one, 1.5)
    two = _beside(T, ended)
    times = []
    for _ in range(4):
        with torch.cuda.stream(two):
            depth.fill_(7)
        two.synchronize()
        t0 = time.monotonic()
        d.bfs(g, ws, 5, depth, None, opts=o, stream=two.cuda_stream)
        times.append(round((time.monotonic() - t0) * 1e3, 2))
        with torch.cuda.stream(two):
            got = depth.cpu().numpy()
        np.testing.assert_array_equal(got, want)
    asleep = not ended.query()
    log(f"searches beside another stream's kernel: {times} ms")
    assert asleep and max(times) < 50 and sum(times[1:]) < 50, times
    ws.destroy()
    g.destroy()
