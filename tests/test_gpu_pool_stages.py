"""The pool's preparation by parts: packed words, rank statistics and, on a
second stream, the region stage, at the edges of their blocks (256 nodes, 8
ranks, 16 ranks in flight).

- the layout of a batch equals, bit for bit, that of each graph prepared in a
  batch of its own and that of a second preparation on another stream;
- the first sweep from the batch's own start is the oracle's, exactly;
- the start lies within 1e-9 of the oracle's (RMS radius, rigid alignment):
  the bound of the FP64 eigen iteration, whose inputs are exact integer sums.
"""
import numpy as np
import pytest

import oracle
from paper_1608_08909_amd import graphs as G
from tests import brute

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


def _prepared(graphs, warm, stream=None):
    pool = ssm.Pool(1 << 28)
    slots = [pool.add(g, k) for g, k in graphs]
    if stream is None:
        pool.prepare(slots, warm=warm)
    else:
        with torch.cuda.stream(stream):
            pool.prepare(slots, warm=warm)
    return pool, slots


@pytest.mark.parametrize("k", [3, 8, 9, 16, 17, 25])
def test_stage_edges(k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    graphs = [(G.rgg(n, n), k) for n in (255, 256, 257, 600)] + [(G.tree_plus(64, 2), k)]
    graphs = [(g, min(k, g.n)) for g, k in graphs]
    p0, s0 = _prepared(graphs, 0)
    p1, s1 = _prepared(graphs, 1)
    p2, s2 = _prepared(graphs, 1, torch.cuda.Stream())
    for q, (g, kq) in enumerate(graphs):
        print("case", g.name, g.n, "k", kq, flush=True)
        ref = oracle.preprocess(g.n, g.row_ptr, g.col_idx, kq)
        assert np.array_equal(p1.export(s1[q], ssm.POOL_REGION), ref.region)
        assert np.array_equal(p1.export(s1[q], ssm.POOL_DEN64), ref.den)
        x0 = p0.export(s0[q], ssm.POOL_X64)
        x1 = p1.export(s1[q], ssm.POOL_X64)
        x1r, _ = oracle.majorize(g.row_ptr, g.col_idx, ref.pivots, ref.dist, ref.wtab, ref.den, x0, 1)
        assert np.array_equal(x1, x1r)
        assert np.array_equal(x1, p2.export(s2[q], ssm.POOL_X64))
        alone, sa = _prepared([graphs[q]], 1)
        assert np.array_equal(x1, alone.export(sa[0], ssm.POOL_X64))
        alone.close()
        w = np.linalg.eigvalsh(oracle.gram(oracle.pmds_center(ref.dist)))[::-1]
        if w[1] > 1e-8 * w[0] and (w[1] - w[2]) / w[0] > 1e-6:  # the plane is unique
            xo, _, _ = oracle.pivotmds(ref.dist)
            xr = oracle.rescale(g.row_ptr, g.col_idx, xo)
            assert brute.coord_error(x0, xr, align=True) < 1e-9
    for p in (p0, p1, p2):
        p.close()
