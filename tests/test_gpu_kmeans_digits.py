"""k-means sp on the 8-bit matrix units: the oracle's clusters, passes and
pivots, bit for bit, for every count of digits and the edges of its tiles."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _check(g, k, max_iters=50):
    print("case", g.name, g.n, "k", k, flush=True)
    piv, dist = oracle.select_pivots(g.n, g.row_ptr, g.col_idx, k, 0)
    ref = oracle.kmeans_sp(dist, piv, max_iters)
    new, assign, passes = ssm.kmeans_pivots(torch.from_numpy(piv).cuda(), torch.from_numpy(dist).cuda(), max_iters)
    assert np.array_equal(new.cpu().numpy(), ref[0])
    assert np.array_equal(assign.cpu().numpy(), ref[1])
    assert passes == ref[2]


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 63, 64, 65, 128, 129, 200])
def test_tiles(k):
    _check(G.rgg(1700, 4), k)


@pytest.mark.parametrize("g,k", [(G.grid(7, 9), 63), (G.path(33), 5), (G.barabasi_albert(3000, 5, 7), 40),
                                 (G.path(300), 20), (G.path(9000), 30), (G.path(40000), 3), (G.tree_plus(4000, 2), 50),
                                 (G.tri_grid(40, 45), 33)],
                         ids=["k=n", "one digit", "ba", "two digits", "long path", "three digits: vector form", "tree", "tri"])
def test_digits(g, k):
    _check(g, k)


@pytest.mark.parametrize("max_iters", [1, 3, 4, 5])
def test_pass_limit(max_iters):
    _check(G.rgg(900, 2), 20, max_iters)
