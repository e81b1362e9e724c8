"""The route a call takes by default is not slower than the one it can be made to
take instead (the faster of several runs of each, with room for their spread)."""
import threading
import time

import numpy as np
import pytest

from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _best(call, reps):
    call()
    times = []
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return min(times)


def _compare(name, call, other, room, reps=4):
    """`other`: the overrides of the other route."""
    own = _best(call, reps)
    with ssm.variants(**other):
        alt = _best(call, reps)
    print("case", name, f"{1e3 * own:.3f} ms, {other}: {1e3 * alt:.3f} ms", flush=True)
    assert own <= room * alt


def _lattice(rows, cols):
    """Triangulated lattice numbered by rows, built on the device."""
    i = torch.arange(rows * cols, device="cuda").reshape(rows, cols)
    u = torch.cat([i[:, :-1].reshape(-1), i[:-1].reshape(-1), i[:-1, :-1].reshape(-1)])
    v = torch.cat([i[:, 1:].reshape(-1), i[1:].reshape(-1), i[1:, 1:].reshape(-1)])
    n = rows * cols
    key = torch.sort(torch.cat([u * n + v, v * n + u])).values
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return ssm.DeviceGraph(n, rp.int(), (key % n).int())


def test_rows_of_a_mesh_too_large_for_the_pages():
    g = _lattice(1900, 1895)
    piv = torch.from_numpy(np.random.default_rng(7).choice(g.n, 40, replace=False).astype(np.int32)).cuda()
    _compare("40 rows", lambda: ssm.bfs_pivots(g, piv), {"bfs_ring": -1}, 1.3)


def test_selections_of_several_threads():
    """Each on a stream of its own: together as fast as on one workgroup each."""
    graphs = [_lattice(300, 300 + q) for q in range(4)]
    streams = [torch.cuda.Stream() for _ in graphs]
    want = [ssm.select_pivots(g, 100) for g in graphs]
    got = [None] * len(graphs)

    def work(q):
        with torch.cuda.stream(streams[q]):
            for _ in range(3):
                got[q] = ssm.select_pivots(graphs[q], 100)

    def all_threads():
        threads = [threading.Thread(target=work, args=(q,)) for q in range(len(graphs))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()

    _compare("4 threads", all_threads, {"select_ahead": -1}, 1.4)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_grid_selection_width():
    """The grid's levels with the rows padded as its lanes want them."""
    g = _lattice(1095, 1095)
    with ssm.variants(select_ahead=-1):
        _compare("grid, k = 8", lambda: ssm.select_pivots(g, 8), {"ell_width": 16}, 1.1, reps=8)


def test_selection_of_few_pivots():
    g = _lattice(300, 300)
    _compare("k = 8", lambda: ssm.select_pivots(g, 8), {"select_ahead": -1}, 1.2, reps=8)


def test_kmeans_of_few_pivots():
    g = _lattice(1000, 1000)
    piv, dist = ssm.select_pivots(g, 3, with_dist=True)
    _compare("k-means, k = 3", lambda: ssm.kmeans_pivots(piv, dist), {"km_chunk": 32}, 1.3)


@pytest.mark.parametrize("count,n,k", [(16, 2500, 50), (64, 5000, 60)])
def test_pool_preparation(count, n, k):
    graphs = [G.rgg(n, q) for q in range(4)]
    pool = ssm.Pool(1 << 32)

    def best(reps=5):
        times = []
        for _ in range(reps):
            slots = [pool.add(graphs[q % 4], k) for q in range(count)]
            torch.cuda.synchronize()
            t = time.perf_counter()
            pool.prepare(slots)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
            for q in slots:
                pool.remove(q)
        return min(times[1:])

    own, alt = best(), []
    for follow in (-1, 1):
        with ssm.variants(pool_follow=follow):
            alt.append(best())
    print("case", count, n, k, [f"{1e3 * t:.3f} ms" for t in [own] + alt], flush=True)
    assert own <= 1.2 * min(alt)
    pool.close()
