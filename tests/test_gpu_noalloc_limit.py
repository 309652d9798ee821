"""The largest graphs that the allocation-free search takes (its 64 MiB of
scratch, counted as noalloc_scratch_bytes does), with few or no delegates: the
last one taken is searched, the next one refused."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda

pytestmark = pytest.mark.gpu

LIMIT = 64 << 20


def _r256(b):
    return (max(b, 256) + 255) // 256 * 256


def _scan(n):
    nb = (n + 2047) // 2048
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    return 256 if nb <= 1 else up(8 * nb) + up(8 * (nb + 1)) + _scan(nb)


def _need(n, d, nds):
    words, dwords = (n + 31) // 32, (d + 31) // 32
    tiles = (((d + 2047) // 2048 + 1) * 8 + 255) // 256 * 256
    return (2 * _r256(4 * words) + 3 * _r256(4 * dwords) + 2 * _r256(4 * n) + 2 * _r256(4 * d) +
            _r256(4 * n) + _r256(8 * (n + 1)) + 2 * _r256(4 * nds) + _r256(_scan(n)) +
            _r256(2 * tiles) + 3328)


@pytest.mark.parametrize("hubs", [0, 3, 2000])
def test_largest_graphs(oracle_mod, hubs):
    d, torch = lib(), torch_cuda()
    leaves = 40 if hubs else 0
    nds = hubs * leaves
    lo, hi = 1 << 20, 1 << 22            # largest n that is taken
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if _need(mid, hubs, nds) <= LIMIT else (lo, mid)
    for n, taken in ((lo, True), (lo - 1, True), (lo + 64, False)):
        # hubs with leaves of their own, one path over the first leaf of each, a
        # path at the end
        v = np.arange(nds, dtype=np.int32)
        src, dst = [n - 1 - nds + v], [n - 1 - hubs - nds + v // max(leaves, 1)]
        end = np.arange(3000, dtype=np.int32)
        src, dst = src + [end], dst + [end + 1]
        if hubs:
            src.append(np.array([3000], np.int32))
            dst.append(np.array([n - 1], np.int32))
            first = n - 1 - nds + leaves * np.arange(hubs, dtype=np.int32)
            src += [first[:-1], np.array([n - 1], np.int32)]
            dst += [first[1:], first[:1]]
        src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
        g = d.Graph(src, dst, n, threshold=32, keep_plain_csr=False)
        st = g.stats
        assert (st["d"], st["n_ndsrc"]) == (hubs, nds)
        depth = torch.full((n,), 5, dtype=torch.int32, device="cuda")
        o = d.run_opts(want_parent=False)
        log(f"noalloc n={n} d={hubs}: needs {_need(n, hubs, nds)} of {LIMIT}")
        if taken:
            d.bfs_noalloc(g, 7, depth, None, opts=o)
            torch.cuda.synchronize()
            want, _ = oracle_mod.Graph(src, dst, n).bfs(7, want_parent=False)
            np.testing.assert_array_equal(depth.cpu().numpy(), want)
        else:
            with pytest.raises(d.DsbfsError) as e:
                d.bfs_noalloc(g, 7, depth, None, opts=o)
            assert e.value.status == d.ERR_RANGE
        g.destroy()
