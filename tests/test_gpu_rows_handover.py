"""Paged BFS rows that cannot be finished as they began: another form gives the
row, with the distances it has always had."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def test_one_way_cycle(forced):
    """A CSR that is not symmetric (the caller's error): the pool is cleared every
    75,000 nodes, so the search comes round to nodes it no longer knows.  It ends
    when it has found more nodes than there are, and the row is the directed one."""
    n, src = 200000, 31
    forced("bfs_ring", 1)
    forced("bfs_pages", 1100)
    rp = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    ci = torch.roll(torch.arange(n, dtype=torch.int32, device="cuda"), -1)
    print("case one-way cycle", n, flush=True)
    dist, _, _ = ssm.bfs_pivots(ssm.DeviceGraph(n, rp, ci), torch.tensor([src], dtype=torch.int32, device="cuda"))
    assert torch.equal(dist[0], (torch.arange(n, device="cuda") - src).remainder(n).int())
