"""The truncated series and the mixing factor on shapes where their kernels
change: the one-work-group form and the general one, every slab width and a
partial last slab, rows around the degree from which a row gets a work group
of its own, L = 0 and 1, and graphs at the small form's largest size. Oracle:
the numpy series and a numpy power iteration in binary64; both sides round a
sum of at most d_max terms per entry and step and P has norm 1, so 1e-11
leaves three digits over L d_max 2^-53 <= 2e-12 (largest case below)."""

import numpy as np
import pytest

from oracle import exact as X
from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu


def hub_graph(n, degrees):
    """A cycle whose first nodes are also joined to many others: hubs of the given degrees."""
    u, v = [np.arange(n)], [np.roll(np.arange(n), -1)]
    for i, d in enumerate(degrees):
        far = (np.arange(d - 2) * 2 + 2 * len(degrees) + 10 + i) % n
        u.append(np.full(far.size, i))
        v.append(far)
    return graphs.csr_from_edges(n, np.concatenate(u), np.concatenate(v))


GRAPHS = {
    "small": lambda: graphs.random_connected(257, 0.05, 3),
    "small_full": lambda: hub_graph(2048, [64, 65, 66, 300]),
    "general": lambda: hub_graph(2049, [63, 64, 65, 257, 800]),
}
_cache = {}


def _graph(key, flags):
    if (key, flags) not in _cache:
        g = _cache.setdefault(key, GRAPHS[key]())
        _cache[(key, flags)] = (g, B.graph_load_csr(g.n, g.row_ptr, g.col, flags))
    return _cache[(key, flags)]


@pytest.mark.parametrize("flags", [B.BD_LAYOUT_CSR, B.BD_LAYOUT_AUTO, B.BD_LAYOUT_FAT | B.BD_RELABEL_DEGREE])
@pytest.mark.parametrize("key", sorted(GRAPHS))
def test_series(key, flags):
    g, dg = _graph(key, flags)
    for Q, L in ((1, 0), (2, 1), (3, 2), (5, 25), (8, 24), (9, 7), (17, 2), (67, 3)):
        s, t = queries.uniform_pairs(g.n, Q, 10 * Q + L)
        s[0], t[0] = 0, g.n - 1  # a hub
        got = B.bd_truncated_beta(dg, s, t, L)
        for i in range(0, Q, 1 + Q // 6):
            assert got[i] == pytest.approx(X.beta_truncated(g, int(s[i]), int(t[i]), L), rel=1e-11), (Q, L, i)


@pytest.mark.parametrize("key", sorted(GRAPHS))
def test_mixing_factor(key):
    g, dg = _graph(key, B.BD_LAYOUT_CSR)
    # the library's iteration, from the same counter-based start vector
    z = (np.uint64(7) + (np.arange(1, g.n + 1, dtype=np.uint64)) * np.uint64(0x9E3779B97F4A7C15))
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    z ^= z >> np.uint64(31)
    y = (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 - 0.5
    rd = np.sqrt(g.deg.astype(np.float64))
    phi = rd / np.linalg.norm(rd)
    A = g.scipy()
    for it in range(41):
        if it:
            y = (A @ (x / rd)) / rd
        y = y - (phi @ y) * phi
        norm = np.linalg.norm(y)
        x = y / norm
        if it in (1, 2, 40):
            assert B.bd_graph_lambda(dg, it, 7) == pytest.approx(norm, rel=1e-11), it
