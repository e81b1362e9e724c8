"""FP64 sweeps of graphs with long rows: the neighbour sums taken by whole
workgroups equal the oracle's, term by term in CSR order, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _hubs(degrees, seed):
    """One hub per degree, its leaves drawn from a common path (so leaves and
    hubs have rows of every kind)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    h = len(degrees)
    n = h + max(degrees) + 50
    i = np.arange(h, n - 1)
    edges = [np.stack([i, i + 1], 1)]
    for q, d in enumerate(degrees):
        leaves = rng.choice(np.arange(h, n), d, replace=False)
        edges.append(np.stack([np.full(d, q), leaves], 1))
    return G.csr_from_edges(n, np.concatenate(edges), "hubs")


@pytest.mark.parametrize("degrees", [(64, 65, 66), (511, 512, 513, 70), (1023, 1024, 1025, 65), (3000, 2049, 100, 64)],
                         ids=lambda d: str(d[0]))
@pytest.mark.parametrize("terms", [0, -1])  # a lane group per node, a thread per node
def test_hub_rows_bit_exact(degrees, terms, forced):
    g = _hubs(degrees, 3)
    k = 7
    print("case", g.n, degrees, terms, flush=True)
    forced("sweep_f64_terms", terms)
    ref = oracle.preprocess(g.n, g.row_ptr, g.col_idx, k)
    dg = ssm.DeviceGraph.from_csr(g)
    piv = ssm.select_pivots(dg, k, 0)
    tm = ssm.build_terms(dg, piv, *ssm.bfs_pivots(dg, piv))
    x0 = np.random.Generator(np.random.PCG64(9)).normal(size=(g.n, 2)) * 5
    x0[g.col_idx[g.row_ptr[1]: g.row_ptr[1] + 40]] = x0[1]  # neighbours of a hub at its place
    for iters in (1, 4):
        xr, _ = oracle.majorize(g.row_ptr, g.col_idx, ref.pivots, ref.dist, ref.wtab, ref.den, x0, iters)
        xg = torch.from_numpy(x0.copy()).cuda()
        ssm.majorize(dg, tm, xg, iters, sync=True)
        assert np.array_equal(xg.cpu().numpy(), xr)
