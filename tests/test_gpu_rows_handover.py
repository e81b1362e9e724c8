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


def _shuffled(g, seed):
    p = np.random.Generator(np.random.PCG64(seed)).permutation(g.n)
    return G.csr_from_edges(g.n, p[g.edges()], g.name + "-shuffled")


def _check(g, piv):
    print("case", g.name, g.n, len(piv), flush=True)
    piv = np.asarray(piv, dtype=np.int32)
    dist, delta, _ = ssm.bfs_pivots(ssm.DeviceGraph.from_csr(g), torch.from_numpy(piv).cuda())
    ref = oracle.bfs_pivots(g.n, g.row_ptr, g.col_idx, piv)
    assert np.array_equal(dist.cpu().numpy(), ref)
    assert np.array_equal(delta.cpu().numpy(), ref.min(0))


LATTICE = G.tri_grid(560, 555)
LEFT = [(LATTICE, 3), (LATTICE, 140), (_shuffled(G.tri_grid(400, 410), 1), 3), (G.tree_plus(200000, 4), 3),
        (G.star(150000), 3)]


@pytest.mark.parametrize("g,k", LEFT, ids=[f"{g.name}-{k}" for g, k in LEFT])
def test_rows_taken_up(g, k, forced):
    """Rows from the middle run out of pages, rows from the corners are called off:
    both are taken up at the level they reached (140 rows: in two chunks)."""
    forced("bfs_ring", 1)
    forced("bfs_pages", 1100)
    _check(g, [g.n // 2 + 280, 0, g.n - 1] + list(range(1000, 1000 + 7 * (k - 3), 7)))


def test_rows_taken_up_by_default():
    """A box lattice: 6 neighbours at most, levels of up to 9,000 nodes."""
    m = 110
    i = np.arange(m ** 3).reshape(m, m, m)
    pairs = [np.stack([a.ravel(), b.ravel()], 1) for a, b in ((i[1:], i[:-1]), (i[:, 1:], i[:, :-1]), (i[..., 1:], i[..., :-1]))]
    _check(G.csr_from_edges(m ** 3, np.concatenate(pairs), "box"), [m ** 3 // 2 + 55, 0] + list(range(5, 5 + 14 * 90001, 90001)))


def _device_csr(n, u, v):
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return ssm.DeviceGraph(n, rp.int(), (key % n).int())


def _lattice(n, cols, hub=0, shuffle=False, diagonals=True):
    """The first n nodes of a triangulated lattice numbered by rows; hub: extra arcs of node n // 2."""
    i = torch.arange(n, device="cuda")
    steps = [(1, i % cols != cols - 1), (cols, i >= 0)] + ([(cols + 1, i % cols != cols - 1)] if diagonals else [])
    ends = [(i[ok & (i + d < n)], (i + d)[ok & (i + d < n)]) for d, ok in steps]
    u, v = torch.cat([a for a, _ in ends]), torch.cat([b for _, b in ends])
    if hub:
        u = torch.cat([u, torch.full((hub,), n // 2, device="cuda")])
        v = torch.cat([v, torch.arange(hub, device="cuda") * 1000])
    if shuffle:
        p = torch.randperm(n, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
        u, v = p[u], p[v]
    return _device_csr(n, u, v)


def _chain(n):
    i = torch.arange(n - 1, device="cuda")
    return _device_csr(n, i, i + 1)


RULE = {  # what the default rule for paged rows looks at, on both sides of its lines
    "15 rows": (lambda: _lattice(1100000, 1051), 15), "16 rows": (lambda: _lattice(1100000, 1051), 16),
    "longest row 8": (lambda: _lattice(1100000, 1051, hub=2), 16), "longest row 9": (lambda: _lattice(1100000, 1051, hub=3), 16),
    "square": (lambda: _lattice(1100000, 1051, diagonals=False), 17), "shuffled": (lambda: _lattice(1100000, 1051, shuffle=True), 16),
    "chain": (lambda: _chain(1090000), 2), "most nodes": (lambda: _lattice(3407488, 1900), 16),
    "one more": (lambda: _lattice(3407489, 1900), 16), "narrow": (lambda: _lattice(1090048, 3), 1),
}


@pytest.mark.parametrize("name", RULE)
def test_rule(name, forced):
    """The default route, the paged form and the other forms give the same rows."""
    make, k = RULE[name]
    g = make()
    piv = torch.linspace(0, g.n - 1, k, device="cuda").long().int()
    print("case", name, g.n, k, flush=True)
    dist = ssm.bfs_pivots(g, piv)[0]
    forced("bfs_ring", -1)
    want = ssm.bfs_pivots(g, piv)[0]
    assert torch.equal(dist, want)
    forced("bfs_ring", 1)
    dist.fill_(7)
    assert torch.equal(ssm.bfs_pivots(g, piv)[0], want)


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
