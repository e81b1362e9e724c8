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
    """Workgroups that wait for the search of a long path see it go on: 60,000
    polls (about 30 ms) are far fewer than its levels take."""
    forced("select_ahead", 4)
    forced("select_m8", state)
    forced("bar_polls", 60000)
    _check(G.path(n), 4)


@pytest.mark.parametrize("state,n", [(0, 41000), (2, 41000), (2, 264000), (3, 264000)])
@pytest.mark.parametrize("cus", [1, 8, 31])
def test_few_compute_units(cus, state, n, forced):
    """Where the searches' workgroups are not resident together, the other forms select."""
    forced("select_ahead", 16)
    forced("select_m8", state)
    forced("ahead_cus", cus)
    _check(G.grid(n // 200, 200), 12)


def _regular(n, seed):
    """Four random cycles: 8 neighbours, and levels that soon hold most nodes."""
    rng = np.random.Generator(np.random.PCG64(seed))
    cycles = [rng.permutation(n) for _ in range(4)]
    return G.csr_from_edges(n, np.concatenate([np.stack([c, np.roll(c, -1)], 1) for c in cycles]), "regular")


def _layers(layers, width, seed):
    """Layers of `width` nodes, three random arcs from each node to the next layer."""
    rng = np.random.Generator(np.random.PCG64(seed))
    u = np.arange((layers - 1) * width)
    v = (u // width + 1)[:, None] * width + rng.integers(0, width, (u.size, 3))
    last = np.stack([np.arange(u.size, u.size + width), u.size - width + np.arange(width)], 1)
    return G.csr_from_edges(layers * width, np.concatenate([np.stack([np.repeat(u, 3), v.ravel()], 1), last]), "layers")


RULE = [(G.grid(205, 200), 95), (G.grid(205, 200), 96), (G.tri_grid(205, 200), 39), (G.tri_grid(205, 200), 40),
        (G.rgg(42000, 3, 8.0), 19), (G.rgg(42000, 3, 8.0), 20), (G.grid(360, 350), 64), (G.tri_grid(360, 350), 48), (G.tri_grid(199, 200), 60),
        (G.barabasi_albert(42000, 5, 2), 30), (G.tree_plus(42000, 5), 120), (_regular(42000, 1), 30),
        (_layers(100, 420, 2), 60), (G.grid(400, 390), 31), (G.grid(400, 390), 32),
        (G.tri_grid(400, 390), 23), (G.tri_grid(400, 390), 24), (G.tri_grid(520, 530), 7),
        (G.tri_grid(520, 530), 8), (G.rgg(280000, 3, 8.0), 8), (_regular(270000, 1), 8)]


@pytest.mark.parametrize("g,k", RULE, ids=[f"{g.name}-{k}" for g, k in RULE])
def test_rule(g, k):
    """Both sides of the default rule's lines, and graphs that leave the form again."""
    _check(g, k)
