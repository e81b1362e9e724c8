"""BFS rows with paged visited bits: the oracle's distances, bit for bit, also
where the pages are taken anew and where they run out and another form steps in."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _check(g, piv):
    print("case", g.name, g.n, flush=True)
    piv = np.asarray(piv, dtype=np.int32)
    dist, delta, region = ssm.bfs_pivots(ssm.DeviceGraph.from_csr(g), torch.from_numpy(piv).cuda())
    ref = oracle.bfs_pivots(g.n, g.row_ptr, g.col_idx, piv)
    assert np.array_equal(dist.cpu().numpy(), ref)
    assert np.array_equal(delta.cpu().numpy(), ref.min(0))


SMALL = [G.path(2), G.path(1000), G.star(300), G.complete(40), G.cycle(1023), G.grid(31, 33), G.tri_grid(60, 70),
         G.tree_plus(3000, 2), G.barabasi_albert(3000, 5, 7), G.rgg(4000, 4)]


@pytest.mark.parametrize("width", [8, 16, 32])
@pytest.mark.parametrize("g", SMALL, ids=[g.name for g in SMALL])
def test_paged_small(g, width, forced):
    forced("bfs_ring", 1)
    forced("ell_width", width)
    _check(g, sorted({0, g.n - 1, g.n // 2}))


def test_paged_pool_taken_anew():
    """The default form above the LDS bits: 10,300 pages pass through a pool of about 7,000."""
    _check(G.tri_grid(1150, 1148), [0, 1150 * 1148 - 1, 660000])


def test_paged_pool_runs_out(forced):
    """A star's second level lies on every page: the other forms give the row."""
    n = 1300000
    forced("bfs_ring", 1)
    g = G.star(n)
    dist, _, _ = ssm.bfs_pivots(ssm.DeviceGraph.from_csr(g), torch.tensor([0, 77], dtype=torch.int32, device="cuda"))
    want = torch.ones(2, n, dtype=torch.int32, device="cuda")
    want[0, 0] = 0
    want[1] = 2
    want[1, 0], want[1, 77] = 1, 0
    assert torch.equal(dist, want)
