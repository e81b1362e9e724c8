"""Max/min selection with searches run ahead of their turn: the same pivots as
the oracle, bit for bit, whatever the graph, the workers and the way a search
keeps its visited set (state bytes, bits, stamps of workgroup groups)."""
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


def _hub(n, hubs, seed):
    """A long path whose nodes also hang on a few hubs of very long rows."""
    rng = np.random.Generator(np.random.PCG64(seed))
    i = np.arange(n - 1)
    leaf = rng.choice(np.arange(hubs, n), n // 3, replace=False)
    return G.csr_from_edges(n, np.concatenate([np.stack([i, i + 1], 1), np.stack([leaf % hubs, leaf], 1)]), f"hub{n}")


SMALL = [
    (G.path(2), 2), (G.path(17), 17), (G.star(70), 9), (G.complete(40), 40), (G.path(900), 12), (G.cycle(1023), 30),
    (G.grid(31, 33), 200), (G.tri_grid(40, 50), 64), (G.tree_plus(3000, 2), 40), (G.barabasi_albert(3000, 5, 7), 60),
    (G.rgg(4000, 4), 120), (_hub(4000, 3, 1), 50), (G.holed_mesh(120, 130, 6, 4, 12, 5), 90),
]


@pytest.mark.parametrize("workers", [1, 3, 8, 16])
@pytest.mark.parametrize("m8", [0, 2])  # state bytes; bits for the pivots after a grid's first BFS
@pytest.mark.parametrize("g,k", SMALL, ids=[g.name for g, _ in SMALL])
def test_ahead_small(g, k, m8, workers, forced):
    forced("select_ahead", workers)
    forced("select_m8", m8)
    _check(g, k)
    _check(g, k, g.n - 1)


@pytest.mark.parametrize("g,k", [(G.grid(200, 203), 40), (G.rgg(42000, 3, 7.0), 60), (G.tree_plus(42000, 5), 20),
                                 (G.barabasi_albert(42000, 5, 2), 20), (G.path(41000), 9), (_hub(45000, 2, 3), 12)],
                         ids=["grid", "rgg", "tree", "ba", "path", "hub"])
@pytest.mark.parametrize("width", [8, 16, 32])
def test_ahead_default_rule(g, k, width, forced):
    """Graphs that keep the form, and wide ones that leave it during or after pivot 0's search."""
    forced("ell_width", width)
    _check(g, k)


@pytest.mark.parametrize("g,k", [(G.grid(500, 530), 24), (G.barabasi_albert(264000, 2, 5), 12)], ids=["grid", "ba"])
@pytest.mark.parametrize("state", [2, 3])  # bits, stamps
@pytest.mark.parametrize("workers", [3, 8])
def test_ahead_after_the_grid(g, k, state, workers, forced):
    forced("select_ahead", workers)
    forced("select_m8", state)
    _check(g, k)


def test_ahead_disconnected(forced):
    g = G.csr_from_edges(43000, np.stack([np.arange(0, 42998), np.arange(1, 42999)], 1), "two parts")
    with pytest.raises(ssm.SSMError) as err:
        ssm.select_pivots(ssm.DeviceGraph.from_csr(g), 10)
    assert err.value.status == ssm.E_DISCONNECTED
