"""PageRank's device memory (scratch and what it keeps with the graph) for all
shares of delegates, against 3 n + 2 d doubles and the columns with a rank for
each delegate; ranks against the oracle (test_gpu_pagerank's tolerance)."""
import numpy as np
import pytest

from gpu_helpers import lib, log, torch_cuda
from test_gpu_build_bytes import _Peak

pytestmark = pytest.mark.gpu


def _graph(n, d, rng):
    """d vertices of degree above 24 among n of a few edges each, shuffled."""
    v = np.arange(n, dtype=np.int64)
    src, dst = [v], [rng.integers(0, n, n)]
    if d:
        src.append(np.repeat(np.arange(d), 40))
        dst.append(rng.integers(0, d if d > 60 else n, 40 * d))
    label = rng.permutation(n)
    return (label[np.concatenate(src)].astype(np.int32), label[np.concatenate(dst)].astype(np.int32))


@pytest.mark.parametrize("share", [0.0, 0.001, 0.2, 0.39, 0.41, 0.6, 0.95, 1.0])
def test_bytes_and_ranks(oracle_mod, share):
    d, torch = lib(), torch_cuda()
    n = 60011
    src, dst = _graph(n, int(share * n), np.random.default_rng(3))
    a = _Peak()
    g = d.Graph(src, dst, n, threshold=24, keep_plain_csr=False, allocator=a)
    st = g.stats
    assert abs(st["d"] / n - share) < 0.02
    held = a.held
    rank = torch.empty(n, dtype=torch.float64, device="cuda")
    O = oracle_mod.Graph(src, dst, n)
    for iters in (1, 2, 12):
        a.peak = a.held
        assert d.pagerank(g, rank, iterations=iters)[0] == iters
        torch.cuda.synchronize()
        np.testing.assert_allclose(rank.cpu().numpy(), O.pagerank(0.85, iters), rtol=1e-10,
                                   atol=1e-18)
        limit = 8 * (3 * n + 2 * st["d"]) + 4 * (st["d"] + st["e_dd"] + st["e_dn"]) + 32768
        log(f"pagerank {st['d']} of {n} delegates: {a.peak - held} of {limit} bytes")
        assert a.peak - held <= limit
    steps, delta = d.pagerank(g, rank, iterations=100, tolerance=1e-7)
    assert 1 < steps < 100 and delta < 1e-7
    np.testing.assert_allclose(rank.cpu().numpy(), O.pagerank(0.85, steps), rtol=1e-10, atol=1e-18)
    g.destroy()
    assert not a.live
