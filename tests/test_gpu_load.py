"""Graph loading on the device: what is refused and what is reported, from host
and from device arrays (every verdict of the host checks), the tables against
the given adjacency through every node's one-step walks, and rows around a
wave's width."""

import numpy as np
import pytest
import torch

from paper_2512_05460_amd import binding as B
from synth import graphs

pytestmark = pytest.mark.gpu

LAYOUTS = [B.BD_LAYOUT_CSR, B.BD_LAYOUT_CSR | B.BD_RELABEL_DEGREE, B.BD_LAYOUT_FAT, B.BD_LAYOUT_COMPACT,
           B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE, B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_WIDE_IDS,
           B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS]


def load(n, rp, col, flags, device):
    if not device:
        return B.graph_load_csr(n, rp, col, flags)
    return B.graph_load_csr_device(n, torch.from_numpy(np.asarray(rp, np.int64)).cuda(),
                                   torch.from_numpy(np.asarray(col, np.int32)).cuda(), flags)


@pytest.mark.parametrize("device", [False, True])
def test_refused(device):
    g = graphs.random_connected(200, 0.04, 1)
    two = graphs.csr_from_edges(8, [0, 1, 2, 4, 5, 6], [1, 2, 0, 5, 6, 7])  # node 3 apart: no edge
    parts = graphs.csr_from_edges(7, [0, 1, 2, 3, 4, 5], [1, 2, 0, 4, 5, 6])

    def broken(edit):
        col = g.col.copy()
        edit(col)
        return g.n, g.row_ptr, col

    r = int(np.flatnonzero(g.deg > 2)[3])
    at = int(g.row_ptr[r])

    def swap(c):
        c[at], c[at + 1] = c[at + 1], c[at]

    def put(v):
        return lambda c: c.__setitem__(at, v)

    missing = next(u for u in range(g.n) if u != r and u not in g.col[at:g.row_ptr[r + 1]] and u < g.col[at + 1])
    cases = [broken(put(-1)), broken(put(g.n)), broken(put(r)), broken(swap), broken(put(int(g.col[at + 1]))),
             broken(put(missing)), (two.n, two.row_ptr, two.col), (parts.n, parts.row_ptr, parts.col)]
    for i, (n, rp, col) in enumerate(cases):
        with pytest.raises(B.ProbeWalkError) as e:
            load(n, rp, col, B.BD_LAYOUT_CSR, device)
        assert e.value.code == B.BD_E_GRAPH, i
    for i in (0, 1):  # ranges are checked without validation too
        with pytest.raises(B.ProbeWalkError) as e:
            load(*cases[i], B.BD_LAYOUT_CSR | B.BD_SKIP_VALIDATION, device)
        assert e.value.code == B.BD_E_GRAPH
    load(*cases[5], B.BD_LAYOUT_CSR | B.BD_SKIP_VALIDATION, device).free()


@pytest.mark.parametrize("device", [False, True])
def test_bipartite(device):
    for g, want in ((graphs.cycle_graph(1000), 1), (graphs.cycle_graph(1001), 0), (graphs.path_graph(2), 1),
                    (graphs.complete_graph(3), 0), (graphs.grid_minus_edges(90, 0.05, 1), 1),
                    (graphs.csr_from_edges(70001, np.zeros(70000, int), np.arange(1, 70001)), 1),
                    (graphs.random_connected(3000, 0.001, 2), 0)):
        dg = load(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR, device)
        info = dg.info()
        assert info["bipartite"] == want and info["n"] == g.n and info["nnz"] == g.nnz, g.name
        assert info["d_min"] == g.d_min and info["d_max"] == g.d_max
        dg.free()


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("flags", LAYOUTS)
def test_tables(flags, device):
    # a hub of 700 neighbours, rows of 63, 64 and 65, and a random remainder
    base = graphs.random_connected(900, 0.01, 9)
    u, v = [np.repeat(np.arange(900), base.deg)], [base.col]
    for i, d in enumerate((700, 63, 64, 65)):
        u.append(np.full(d, i))
        v.append(np.arange(900 - d, 900))
    g = graphs.csr_from_edges(900, np.concatenate(u), np.concatenate(v))
    dg = load(g.n, g.row_ptr, g.col, flags, device)
    # every node's first steps, for several draws of the neighbour
    start = np.tile(np.arange(g.n), 40)
    p = np.repeat(np.arange(40), g.n)
    tr, _ = B.bd_walk_trace(dg, start, 1, 2, p, 0, 2, 77)
    ref = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR)
    want, _ = B.bd_walk_trace(ref, start, 1, 2, p, 0, 2, 77)
    assert np.array_equal(tr, want)
    for a, b in ((0, 1), (1, 2)):  # and each is an edge of the graph
        key = tr[:, a].astype(np.int64) * g.n + tr[:, b]
        assert np.isin(key, np.repeat(np.arange(g.n, dtype=np.int64), g.deg) * g.n + g.col).all()
    dg.free()
    ref.free()


@pytest.mark.parametrize("close", [None, 0, 1])
@pytest.mark.parametrize("seed", [1, 2])
def test_long_chains(seed, close):
    """Paths with shuffled ids and their cycles (long climbs in the union-find,
    no hub to hang under), and the same with one edge left out."""
    n = 40000 + (close or 0)
    p = np.random.default_rng(seed).permutation(n)
    u, v = p[:-1], p[1:]
    if close is not None:
        u, v = np.append(u, p[-1]), np.append(v, p[0])
    g = graphs.csr_from_edges(n, u, v)
    dg = load(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR, False)
    assert dg.info()["bipartite"] == (0 if close == 1 else 1)
    dg.free()
    cut = np.ones(u.size, bool)
    cut[n // 3] = False
    if close is not None:
        cut[n // 2] = False
    g = graphs.csr_from_edges(n, u[cut], v[cut])
    with pytest.raises(B.ProbeWalkError) as e:
        load(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR, False)
    assert e.value.code == B.BD_E_GRAPH
