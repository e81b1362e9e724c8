"""The FP32 sweep's launch shapes timed on a loop's own sweeps: the loop's
result equals, bit for bit, that of a loop without any timing, whether its
sweeps suffice for all shapes (131, 132: an odd and an even count, no sweep
lost or run twice), do not (24: copies), or a stop test is on (copies); and so
does the next loop on the same graph, with the plan kept."""
import numpy as np
import pytest

from paper_1608_08909_amd import graphs as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1608_08909_amd import ssm


@pytest.mark.parametrize("family", ["rgg", "ba", "grid"])
@pytest.mark.parametrize("iters,tol", [(24, 0.0), (131, 0.0), (132, 0.0), (131, 1e-3)])
def test_tuned_loop_is_the_untimed_loop(family, iters, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    q = iters + (7 if tol else 0)  # a graph shape of its own: the first loop on it is timed
    g = {"rgg": lambda: G.rgg(20000 + q, 5), "ba": lambda: G.barabasi_albert(3000 + q, 5, 7),
         "grid": lambda: G.grid(40, 20 + q)}[family]()
    k = 33
    print("case", g.name, g.n, iters, tol, flush=True)
    dg = ssm.DeviceGraph.from_csr(g)
    piv = ssm.select_pivots(dg, k, 0)
    terms = ssm.build_terms(dg, piv, *ssm.bfs_pivots(dg, piv))
    x0 = ssm.pivotmds_init(dg, terms, ssm.FP32)
    ssm.set_variant("sweep_tune", -1)
    try:
        ref = x0.clone()
        want = ssm.majorize(dg, terms, ref, iters, tol=tol, sync=True)
    finally:
        ssm.set_variant(None)
    for _ in range(2):
        x = x0.clone()
        assert ssm.majorize(dg, terms, x, iters, tol=tol, sync=True) == want
        assert torch.equal(x, ref)
    assert np.isfinite(ref.cpu().numpy()).all()
