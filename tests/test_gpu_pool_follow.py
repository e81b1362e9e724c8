"""The pool's BFS beside its selections: the same pivots, distances and
failures as with the BFS after them, for the smallest and the largest batch
that takes the form (one graph, one per compute unit), one graph more, and a
batch with disconnected graphs first, in the middle and last."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _batch(count, broken):
    mix = [(G.grid(7, 9), 6), (G.path(300), 3), (G.tree_plus(900, 2), 33), (G.rgg(1500, 4), 17),
           (G.grid(50, 50), 50), (G.star(40), 3), (G.holed_mesh(60, 65, 3, 4, 8, 5), 40)]
    out = [mix[q % len(mix)] for q in range(count)]
    bad = G.csr_from_edges(9, np.array([[0, 1], [1, 2], [3, 4], [4, 5], [6, 7], [7, 8]]))
    for q in broken:
        out[q] = (bad, 5)
    return out


@pytest.mark.parametrize("extra,broken", [(None, []), (9, [0, 4, 8]), (0, []), (1, [])])
def test_follow(extra, broken):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    count = 1 if extra is None else extra if broken else cus + extra
    graphs = _batch(count, broken)
    refs = {}
    for follow in (0, -1):
        print("case", count, broken, "pool_follow", follow, flush=True)
        ssm.set_variant("pool_follow", follow)
        try:
            pool = ssm.Pool(1 << 30)
            slots = [pool.add(g, k) for g, k in graphs]
            pool.prepare(slots)
        finally:
            ssm.set_variant("pool_follow", 0)
        for q, (g, k) in enumerate(graphs):
            info = pool.info(slots[q])
            if q in broken:
                assert info["state"] == ssm.POOL_FAILED and info["fail"] == ssm.E_DISCONNECTED
                continue
            assert info["state"] == ssm.POOL_READY
            if (g.name, k) not in refs:
                refs[g.name, k] = oracle.preprocess(g.n, g.row_ptr, g.col_idx, k)
            ref = refs[g.name, k]
            assert np.array_equal(pool.export(slots[q], ssm.POOL_PIVOTS), ref.pivots)
            assert np.array_equal(pool.export(slots[q], ssm.POOL_DIST), ref.dist)
            assert info["dmax"] == ref.dmax
        pool.close()
