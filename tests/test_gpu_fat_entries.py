"""The fat layout's two entry sizes (8 bytes up to degree 127, 16 above) against
the oracle, bit for bit: walks too short for sign tables, walk sharing, recorded
paths' end points, and the highest degree of each size."""

import numpy as np
import pytest

from oracle import estimator as E
from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu

SEED = graphs.PHILOX_SEED


def wheel(spokes):
    i = np.arange(1, spokes + 1)
    u = np.concatenate([np.zeros(spokes, int), i, [spokes], np.arange(spokes + 1, spokes + 4000)])
    v = np.concatenate([i, np.roll(i, -1), [spokes + 1], np.arange(spokes + 2, spokes + 4001)])
    return graphs.csr_from_edges(spokes + 4001, u, v)


@pytest.mark.parametrize("spokes", [127, 128])
@pytest.mark.parametrize("R,M", [(3, 1), (50, 1), (3, 2), (50, 4)])
def test_entries(spokes, R, M):
    g = wheel(spokes)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_FAT)
    assert dg.info()["d_max"] == spokes and dg.info()["layout"] == 1
    s, t = queries.uniform_pairs(spokes, 3, R)
    L = np.array([1, 6, 31], np.int32)
    uid = np.arange(3) + 3
    ref = E.estimate(g, s, t, L, [(3, 37, 111, R)] * 3, SEED, uid=uid, threads=8, share=M)
    for mode in ("plain", "batched"):
        got = B.bd_query_batch(dg, s, t, 0.1, L, SEED, B.policy("fixed", B=3, R=R, share=M), B.exec_cfg(mode), uid=uid)
        assert np.all(got["status"] == 0) and np.array_equal(got["beta"], ref), mode
    dg.free()


@pytest.mark.parametrize("spokes", [127, 128])
def test_recorded_paths(spokes):
    g = wheel(spokes)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_FAT)
    start = np.array([0, spokes, spokes + 1, g.n - 1], np.int32)
    tr, acc = B.bd_walk_trace(dg, start, 5, 2, np.arange(4), [0, 1, 0, 1], 61, SEED)
    for i in range(4):
        path, total = E.walk_trace(g, int(start[i]), 61, SEED, 5, 2, i, i & 1)
        assert np.array_equal(tr[i], path) and acc[i] == np.float32(total)
    dg.free()


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1])
def test_most_nodes_of_small_entries(n):
    g = graphs.cycle_graph(n)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_FAT)
    s, t = np.array([n - 1, n - 3, n // 2], np.int32), np.array([n - 2, 1, n - 1], np.int32)
    uid = np.arange(3) + 3
    ref = E.estimate(g, s, t, 50, [(3, 37, 111, 40)] * 3, SEED, uid=uid, threads=8, share=1)
    for mode in ("plain", "batched"):
        got = B.bd_query_batch(dg, s, t, 0.1, 50, SEED, B.policy("fixed", B=3, R=40), B.exec_cfg(mode), uid=uid)
        assert np.all(got["status"] == 0) and np.array_equal(got["beta"], ref), mode
    dg.free()


def test_last_offsets_of_small_entries():
    """Row offsets of 8-byte entries go to within 2% of 2^32 bytes: 2^22 nodes in a ring,
    each joined to its 63 nearest on either side; the 16-byte entries' results."""
    import torch
    n, k = 1 << 22, 63
    off = torch.cat([torch.arange(-k, 0), torch.arange(1, k + 1)]).to(device="cuda", dtype=torch.int32)
    col = torch.arange(n, device="cuda", dtype=torch.int32)[:, None] + off
    col[:k] %= n
    col[-k:] %= n
    col[:k], col[-k:] = col[:k].sort(1).values, col[-k:].sort(1).values
    rp = torch.arange(n + 1, device="cuda", dtype=torch.int64) * (2 * k)
    s, t = np.array([n - 1, n - 200, 5], np.int32), np.array([n - 2, 3, n - 70], np.int32)
    got = {}
    for name, flag in (("8", B.BD_TEMPORAL), ("16", B.BD_NONTEMPORAL)):
        dg = B.graph_load_csr_device(n, rp, col.reshape(-1), B.BD_LAYOUT_FAT | flag | B.BD_SKIP_VALIDATION)
        assert dg.info()["d_max"] == 2 * k and dg.info()["nontemporal"] == (name == "16")
        got[name] = B.bd_query_batch(dg, s, t, 0.1, 80, SEED, B.policy("fixed", B=3, R=40), B.exec_cfg("batched"))
        dg.free()
    assert np.all(got["8"]["status"] == 0) and np.array_equal(got["8"]["beta"], got["16"]["beta"])
