"""The pool's BFS beside its selections, forced on small batches: the oracle's
pivots and distances, whichever way the batch goes."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm

MIX = [(G.grid(7, 9), 6), (G.path(300), 3), (G.tree_plus(900, 2), 33), (G.rgg(1500, 4), 17), (G.star(40), 3)]
BAD = G.csr_from_edges(9, np.array([[0, 1], [1, 2], [3, 4], [4, 5], [6, 7], [7, 8]]))


@pytest.mark.parametrize("follow", [0, 1, -1])
@pytest.mark.parametrize("count,broken", [(1, []), (2, [0]), (9, [0, 4, 8]), (60, [])])
def test_small_batches(count, broken, follow, forced):
    print("case", count, broken, "pool_follow", follow, flush=True)
    forced("pool_follow", follow)
    graphs = [(BAD, 5) if q in broken else MIX[q % len(MIX)] for q in range(count)]
    pool = ssm.Pool(1 << 29)
    slots = [pool.add(g, k) for g, k in graphs]
    pool.prepare(slots)
    refs = {}
    for q, (g, k) in enumerate(graphs):
        info = pool.info(slots[q])
        if q in broken:
            assert info["state"] == ssm.POOL_FAILED and info["fail"] == ssm.E_DISCONNECTED
            continue
        assert info["state"] == ssm.POOL_READY
        if g.name not in refs:
            refs[g.name] = oracle.preprocess(g.n, g.row_ptr, g.col_idx, k)
        assert np.array_equal(pool.export(slots[q], ssm.POOL_PIVOTS), refs[g.name].pivots)
        assert np.array_equal(pool.export(slots[q], ssm.POOL_DIST), refs[g.name].dist)
        assert info["dmax"] == refs[g.name].dmax
    pool.close()
