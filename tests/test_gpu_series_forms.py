"""The truncated series on both sides of the rules that choose its form: dense small
graphs (one work group, or the general form), and the number of rows from which a
row has fewer lanes than a wave, for every slab width; long series. Oracle: the
numpy series in binary64. A step rounds a sum of at most d_max terms per entry on
both sides and P has norm 1: L d_max 2^-53."""

import numpy as np
import pytest

from oracle import exact as X
from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu

EDGE = 8000  # rows of all slabs


def _check(g, dg, Q, L):
    s, t = queries.uniform_pairs(g.n, Q, Q + L)
    got = B.bd_truncated_beta(dg, s, t, L)
    for i in range(0, Q, 1 + Q // 3):
        ref = X.beta_truncated(g, int(s[i]), int(t[i]), L)
        assert got[i] == pytest.approx(ref, rel=(L + 1) * max(g.deg.max(), 16) * 2.0 ** -52), (g.n, Q, L, i)


@pytest.mark.parametrize("n", [EDGE // 4, EDGE // 4 + 1, EDGE, EDGE + 1])
@pytest.mark.parametrize("flags", [B.BD_LAYOUT_CSR, B.BD_LAYOUT_AUTO])
def test_lanes_of_a_row(n, flags):
    i = np.arange(n)
    far = np.random.default_rng(n).integers(0, n, 3 * n)
    u, v = np.concatenate([i[1:], np.repeat(i, 3), np.zeros(90, int)]), np.concatenate([i[:-1], far, far[:90]])
    g = graphs.csr_from_edges(n, u[u != v], v[u != v])  # a hub of degree above 64
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    for Q, L in ((1, 40), (2, 3), (3, 40), (7, 40), (16, 3), (17, 3), (40, 40), (64, 300)):
        _check(g, dg, Q, L)
    dg.free()


@pytest.mark.parametrize("n,p", [(250, 0.9), (1000, 0.03), (1000, 0.004), (2048, 0.01)])
def test_dense_and_sparse_small_graphs(n, p):
    g = graphs.random_connected(n, p, 3)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR)
    for Q, L in ((1, 2000), (5, 40), (64, 200), (300, 40)):
        _check(g, dg, Q, L)
    dg.free()
