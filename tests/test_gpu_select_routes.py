"""Selection with searches ahead: the rules that choose it and its limits."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _check(g, k, first=0):
    print("case", g.name, g.n, "k", k, flush=True)
    piv, _ = oracle.select_pivots(g.n, g.row_ptr, g.col_idx, k, first)
    got = ssm.select_pivots(ssm.DeviceGraph.from_csr(g), k, first).cpu().numpy()
    assert np.array_equal(got, piv)


@pytest.mark.parametrize("n,state", [(120000, 0), (200000, 0), (263000, 2), (263000, 3)],
                         ids=["bytes", "bits", "bits after the grid", "stamps"])
def test_a_search_longer_than_the_barrier_waits(n, state, forced):
    """Workgroups that wait for the search of a long path see it go on: 30,000
    polls (about 20 ms) are far fewer than its levels take."""
    forced("select_ahead", 4)
    forced("select_m8", state)
    forced("bar_polls", 30000)
    _check(G.path(n), 4)


@pytest.mark.parametrize("state,n", [(0, 41000), (2, 41000), (2, 264000), (3, 264000)])
@pytest.mark.parametrize("cus", [1, 8, 31])
def test_few_compute_units(cus, state, n, forced):
    """Where the searches' workgroups are not resident together, the other forms select."""
    forced("select_ahead", 16)
    forced("select_m8", state)
    forced("ahead_cus", cus)
    _check(G.grid(n // 200, 200), 12)
