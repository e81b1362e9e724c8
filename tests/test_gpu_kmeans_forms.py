"""k-means sp: the form taken at each number of pivots, and the matrix form at the
digit counts and tile edges it is built for, against the oracle bit for bit."""
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


@pytest.mark.parametrize("k", [47, 48, 49])
def test_rule(k):
    _check(G.rgg(1700, 4), k)


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 33])
def test_matrix_form_of_few_pivots(k, forced):
    forced("km_matrix", 1)
    _check(G.rgg(1700, 4), k)


@pytest.mark.parametrize("form", [1, -1])
@pytest.mark.parametrize("n,leaves,most", [(2000, 0, 3), (9000, 0, 4), (31000, 2, 5)])
def test_sum_digits(n, leaves, most, form, forced):
    """A path with leaves on its nodes: n (leaves + 1) times the largest distance takes `most` digits."""
    i = np.arange(n)
    arms = [np.stack([i, n + leaves * i + q], 1) for q in range(leaves)]
    g = G.csr_from_edges(n * (leaves + 1), np.concatenate([np.stack([i[:-1], i[1:]], 1)] + arms), f"arms{n}")
    top = float(g.n) * (n - 1 + (2 if leaves else 0))
    digits = [q for q in range(2, 8) if top <= 127 * (256 ** q - 1) // 255][0]
    assert digits == most
    forced("km_matrix", form)
    _check(g, 3, 12)
