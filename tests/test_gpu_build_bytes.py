"""The most device memory a build holds at a time, through an allocator that
counts: edge lists that are mostly loops (which the keys need no room for), few
edges on many vertices, many edges; from the host and on the device, with and
without the plain rows. The limits are what builds held at most before the
builder packed its pairs in blocks."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda
from test_gpu_alloc_failure import CountingAllocator

pytestmark = pytest.mark.gpu

N = 1 << 18


class _Peak(CountingAllocator):
    def __init__(self):
        super().__init__()
        self.held = self.peak = 0
        alloc, free, d = self._a, self._f, lib()

        def _alloc(ctx, nbytes, stream):
            p = alloc(ctx, nbytes, stream)
            self.held += nbytes
            self.peak = max(self.peak, self.held)
            return p

        def _free(ctx, ptr, stream):
            self.held -= self.live.get(ptr, 0)
            free(ctx, ptr, stream)

        self._keep = alloc, free
        self._a, self._f = d.ALLOC_FN(_alloc), d.FREE_FN(_free)
        self.struct = d.dsbfs_allocator(None, self._a, self._f)


def _edges(kind):
    rng = np.random.default_rng(8)
    if kind == "few":
        return (rng.integers(0, N, 100, dtype=np.int32) for _ in range(2))
    u = rng.integers(0, N, 8 * N, dtype=np.int32)
    v = rng.integers(0, N, 8 * N, dtype=np.int32)
    if kind == "loops":
        v[:8 * N * 15 // 16] = u[:8 * N * 15 // 16]
    elif kind == "only loops":
        v = u.copy()
    return u, v


# bytes a vertex
@pytest.mark.parametrize("kind,plain,device,limit", [
    ("few", False, False, 47.1), ("few", True, True, 47.1),
    ("loops", False, False, 80.2), ("loops", False, True, 59.1), ("loops", True, True, 66.1),
    ("only loops", True, False, 64.2), ("only loops", True, True, 47.1),
    ("edges", False, True, 264.1), ("edges", True, False, 495.1)])
def test_build_peak(oracle_mod, kind, plain, device, limit):
    d, torch = lib(), torch_cuda()
    src, dst = _edges(kind)
    a = _Peak()
    to = (lambda x: torch.from_numpy(x).cuda()) if device else (lambda x: x)
    g = d.Graph(to(src), to(dst), N, threshold=32, keep_plain_csr=plain, allocator=a)
    log(f"{kind} plain={plain} device={device}: {a.peak / N:.2f} of {limit} bytes a vertex")
    O = oracle_mod.Graph(src, dst, N)
    np.testing.assert_array_equal(g.export(0, np.int32), O.degrees())
    assert a.peak <= limit * N
    # an endpoint outside the range is refused before the keys are allocated
    bad = dst.copy()
    bad[len(bad) // 2] = N
    b = _Peak()
    with pytest.raises(d.DsbfsError) as e:
        d.Graph(to(src), to(bad), N, threshold=32, keep_plain_csr=plain, allocator=b)
    assert e.value.status == d.ERR_INVALID_ARG
    assert not b.live and b.peak <= (0 if device else 8 * len(src)) + 4096
    g.destroy()
    assert not a.live
