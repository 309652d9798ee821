"""Searches and batches that want the compute units at the same time: a batch
(whose grid needs all of them) is served beside searches that never pause, and
beside kernels of other streams; nobody waits for work that another caller's
stream still has to do first."""
import threading
import time

import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda

pytestmark = pytest.mark.gpu


class _Setup:
    def __init__(self, inputs_mod, oracle_mod, scale=18, k=6):
        self.d = lib()
        self.torch = torch_cuda()
        self.probe = self.torch.zeros(1, device="cuda")
        self.n = 1 << scale
        src, dst = inputs_mod.rmat_edges(scale)
        self.g = self.d.Graph(src, dst, self.n, threshold=32)
        O = oracle_mod.Graph(src, dst, self.n)
        self.sources = inputs_mod.pick_sources(src, dst, self.n, k, seed=11).tolist()
        self.want = {s: O.bfs(s, want_parent=False)[0] for s in self.sources}

    def search(self, ws, depth, stream, s):
        self.d.bfs(self.g, ws, s, depth, None, opts=self.d.run_opts(want_parent=False),
                   stream=stream.cuda_stream)

    def batch(self, ws, depth, stream):
        self.d.msbfs(self.g, ws, self.sources, depth, stream=stream.cuda_stream)

    def rows_right(self, depth):
        got = depth.cpu().numpy()
        return all(np.array_equal(got[i], self.want[s]) for i, s in enumerate(self.sources))


def test_batches_are_served_beside_searches_without_pause(inputs_mod, oracle_mod):
    """Two threads whose searches last a quarter of a second (a path: a barrier
    or two for each of 30000 levels) and follow one another without a pause, so
    that compute units are taken at nearly every moment, and two threads with
    batches. The searches go on until every batch has returned, or until a limit
    that only batches never served would reach."""
    T = _Setup(inputs_mod, oracle_mod, scale=14)
    d, torch, limit, n = T.d, T.torch, 12.0, 30000
    v = np.arange(n - 1, dtype=np.int32)
    path = d.Graph(v, v + 1, n, threshold=32, keep_plain_csr=False)
    batches_done, errors, bad, count = threading.Event(), [], [], [0, 0]
    t0 = time.monotonic()

    def searches(k):
        try:
            stream, ws = torch.cuda.Stream(), d.Workspace(path)
            depth = torch.empty(n, dtype=torch.int32, device="cuda")
            time.sleep(0.1 * k)
            while not batches_done.is_set() and time.monotonic() - t0 < limit:
                d.bfs(path, ws, 0, depth, None, opts=d.run_opts(want_parent=False),
                      stream=stream.cuda_stream)
                count[k] += 1
            if not np.array_equal(depth.cpu().numpy(), np.arange(n)):
                bad.append(k)
        except Exception as e:
            errors.append(e)

    def batches():
        try:
            stream, ws = torch.cuda.Stream(), d.Workspace(T.g, max_lanes=64)
            depth = torch.empty((len(T.sources), T.n), dtype=torch.int32, device="cuda")
            for i in range(3):
                T.batch(ws, depth, stream)
                if not T.rows_right(depth):
                    bad.append(("batch", i))
        except Exception as e:
            errors.append(e)

    searchers = [threading.Thread(target=searches, args=(k,)) for k in range(2)]
    for t in searchers:
        t.start()
    while min(count) < 2 and not errors:  # both are at it, their first calls behind them
        time.sleep(0.01)
    start = time.monotonic()
    batchers = [threading.Thread(target=batches) for _ in range(2)]
    for t in batchers:
        t.start()
    for t in batchers:
        t.join()
    took = time.monotonic() - start
    batches_done.set()
    for t in searchers:
        t.join()
    log(f"6 batches beside {sum(count)} searches in {took:.2f} s")
    assert not errors, errors
    assert not bad, bad
    assert took < limit / 2, f"batches took {took:.1f} s: served only once the searches had ended"
    path.destroy()
    T.g.destroy()


def _sleep(T, stream, seconds):
    """Puts a kernel of one wave on stream that runs for at least `seconds`, up to
    about three times as long; the event recorded after it. (It counts cycles of
    a clock that rises under load: the rate is the highest of a few short ones,
    twice over.)"""
    torch = T.torch
    with torch.cuda.stream(stream):
        best = None
        for _ in range(6):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            torch.cuda._sleep(50_000_000)
            e1.record()
            e1.synchronize()
            best = min(best or 1e9, e0.elapsed_time(e1))
        torch.cuda._sleep(int(50_000_000 * 2 * seconds * 1e3 / best))
        ended = torch.cuda.Event()
        ended.record()
    return ended


def _beside(T, ended):
    """A stream whose kernels run beside the one that `ended` comes after. (The
    runtime has four hardware queues, and streams that share one wait for each
    other, which no library call on them can change.)"""
    torch = T.torch
    for _ in range(8):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            T.probe.add_(1)
            done = torch.cuda.Event()
            done.record()
        until = time.monotonic() + 0.05
        while time.monotonic() < until and not done.query():
            time.sleep(0.001)
        if done.query():
            assert not ended.query()
            return stream
        log("a stream shares the long kernel's hardware queue")
    pytest.fail("no stream runs beside the long kernel")


def test_batch_beside_another_streams_kernel(inputs_mod, oracle_mod):
    """A batch of one word starts while another stream's kernel of a single wave
    runs: its blocks leave that wave's compute unit room."""
    T = _Setup(inputs_mod, oracle_mod, scale=14)
    torch = T.torch
    ws = T.d.Workspace(T.g, max_lanes=64)
    rows = torch.empty((len(T.sources), T.n), dtype=torch.int32, device="cuda")
    one = torch.cuda.Stream()
    T.batch(ws, rows, one)  # what only a first call does
    rows.fill_(7)
    torch.cuda.synchronize()
    ended = _sleep(T, one, 0.7)
    two = _beside(T, ended)
    t0 = time.monotonic()
    T.batch(ws, rows, two)
    took = time.monotonic() - t0
    asleep = not ended.query()
    log(f"batch beside another stream's kernel: {took * 1e3:.1f} ms")
    assert T.rows_right(rows)
    assert asleep, f"the batch returned only after the other stream's kernel ({took:.2f} s)"
    T.g.destroy()


@pytest.mark.parametrize("queued", ["search", "batch"])
def test_no_wait_for_earlier_work_of_another_stream(inputs_mod, oracle_mod, queued):
    """A call queued behind a long kernel of its own stream does not keep a batch
    on another stream waiting until that kernel has ended."""
    T = _Setup(inputs_mod, oracle_mod, scale=16)
    d, torch = T.d, T.torch
    ws, wb, wc = d.Workspace(T.g), *(d.Workspace(T.g, max_lanes=64) for _ in range(2))
    depth = torch.empty(T.n, dtype=torch.int32, device="cuda")
    rows, rows_c = (torch.empty((len(T.sources), T.n), dtype=torch.int32, device="cuda")
                    for _ in range(2))
    one = torch.cuda.Stream()
    T.search(ws, depth, one, T.sources[0])  # what only first calls do
    T.batch(wc, rows_c, one)
    T.batch(wb, rows, one)
    rows.fill_(7)
    torch.cuda.synchronize()
    ended = _sleep(T, one, 0.9)
    two = _beside(T, ended)
    errors = []

    def behind():
        try:
            if queued == "search":
                T.search(ws, depth, one, T.sources[1])
            else:
                T.batch(wc, rows_c, one)
        except Exception as e:
            errors.append(e)

    t = threading.Thread(target=behind)
    t.start()
    time.sleep(0.1)
    t0 = time.monotonic()
    T.batch(wb, rows, two)
    took = time.monotonic() - t0
    asleep = not ended.query()
    t.join()
    log(f"batch beside a {queued} behind a long kernel: {took * 1e3:.1f} ms")
    assert not errors, errors
    assert T.rows_right(rows) and T.rows_right(rows_c)
    assert np.array_equal(depth.cpu().numpy(), T.want[T.sources[int(queued == "search")]])
    assert asleep, f"the batch returned only after the other stream's kernel ({took:.2f} s)"
    T.g.destroy()
