"""The route a call takes by default is not slower than the one it can be made to
take instead (the faster of several runs of each, with room for their spread)."""
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
    _compare("40 rows", lambda: ssm.bfs_pivots(g, piv), {"bfs_ring": -1}, 1.15)
