"""FP64 sweeps over a graph whose long rows are not those the terms were built
for (same node and arc counts, which is all that a call can check): the terms'
weights with the given graph's neighbours, as on every graph without long rows."""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm

N, EXTRA = 1200, 300


def _chain(extra, name):
    i = np.arange(N - 1)
    return G.csr_from_edges(N, np.concatenate([np.stack([i, i + 1], 1), extra]), name)


def _hub(at):
    far = np.array([q for q in range(N) if abs(q - at) > 1])[: 3 * EXTRA: 3]
    return _chain(np.stack([np.full(EXTRA, at), far], 1), f"hub{at}")


FLAT = _chain(np.stack([np.arange(EXTRA) * 2, np.arange(EXTRA) * 2 + 500], 1), "no hub")


@pytest.mark.parametrize("terms", [0, -1])  # a lane group per node, a thread per node
@pytest.mark.parametrize("built,given", [(_hub(0), _hub(700)), (FLAT, _hub(700)), (_hub(5), FLAT)],
                         ids=["other hub", "hub not listed", "hub gone"])
def test_long_rows_of_another_graph(built, given, terms, forced):
    print("case", built.name, given.name, terms, flush=True)
    assert built.nnz == given.nnz
    forced("sweep_f64_terms", terms)
    k = 7
    ref = oracle.preprocess(built.n, built.row_ptr, built.col_idx, k)
    dg = ssm.DeviceGraph.from_csr(built)
    piv = ssm.select_pivots(dg, k, 0)
    tm = ssm.build_terms(dg, piv, *ssm.bfs_pivots(dg, piv))
    x0 = np.random.Generator(np.random.PCG64(9)).normal(size=(N, 2)) * 5
    xr, _ = oracle.majorize(given.row_ptr, given.col_idx, ref.pivots, ref.dist, ref.wtab, ref.den, x0, 3)
    xg = torch.from_numpy(x0.copy()).cuda()
    ssm.majorize(ssm.DeviceGraph.from_csr(given), tm, xg, 3, sync=True)
    assert np.array_equal(xg.cpu().numpy(), xr)
