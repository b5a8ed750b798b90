"""The sign-table walk kernels against the oracle, bit for bit: both forms
(adjacency in LDS, and three-byte positions read from memory), replica counts
around a wave and around the wave-uniform rule, lengths with every remainder
of four, walk sharing, split probes, both sides of the rule that chooses
them, and endpoints of extreme degree. A binary64 result is compared for
equality: sums are exact integers, so the order of work cannot show."""

import numpy as np
import pytest

from oracle import estimator as E
from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu

SEED = graphs.PHILOX_SEED
STORAGE = B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS
LAYOUTS = [B.BD_LAYOUT_CSR, B.BD_LAYOUT_AUTO, B.BD_LAYOUT_FAT, STORAGE]


def wheel(n):
    """A hub joined to every node of a cycle: degrees n - 1 and 3."""
    i = np.arange(1, n)
    return graphs.csr_from_edges(n, np.concatenate([np.zeros(n - 1, int), i]), np.concatenate([i, np.roll(i, -1)]))


GRAPHS = {  # in LDS, in LDS with one run of degrees, in memory (96,000 entries), in memory with a hub of degree 40,000
    "small": lambda: graphs.random_connected(300, 0.03, 5),
    "cycle": lambda: graphs.cycle_graph(1001),
    "dense": lambda: graphs.random_connected(1600, 0.0375, 6),
    "wheel": lambda: wheel(40001),
}
_cache = {}


def _graph(key, flags):
    if (key, flags) not in _cache:
        g = _cache.setdefault(key, GRAPHS[key]())
        _cache[(key, flags)] = (g, B.graph_load_csr(g.n, g.row_ptr, g.col, flags))
    return _cache[(key, flags)]


def _check(key, flags, s, t, L, Bb, R, M=1, modes=("plain", "batched"), **kw):
    g, dg = _graph(key, flags)
    ref_g, rs, rt = g, s, t
    if flags == STORAGE:
        ref_g, _, internal = graphs.storage_order(g)
        rs, rt = internal[s], internal[t]
    uid = np.arange(len(s)) + 3
    ref = E.estimate(ref_g, rs, rt, L, [(Bb, 37, Bb * 37, R)] * len(s), SEED, uid=uid, threads=8, share=M)
    for mode in modes:
        got = B.bd_query_batch(dg, s, t, 0.1, L, SEED, B.policy("fixed", B=Bb, R=R, share=M), B.exec_cfg(mode, **kw),
                               uid=uid)
        assert np.all(got["status"] == 0) and np.array_equal(got["beta"], ref), (key, flags, L, Bb, R, M, mode)


@pytest.mark.parametrize("flags", LAYOUTS)
@pytest.mark.parametrize("key", ["small", "cycle", "dense"])
@pytest.mark.parametrize("R,L", [(47, 33), (48, 32), (64, 31), (65, 30), (130, 13)])
def test_replicas_and_lengths(key, flags, R, L):
    g, _ = _graph(key, flags)
    s, t = queries.uniform_pairs(g.n, 3, R)
    _check(key, flags, s, t, L, 3, R)


@pytest.mark.parametrize("key", ["small", "dense"])
@pytest.mark.parametrize("M", [2, 3, 4])
def test_sharing(key, M):
    s, t = queries.uniform_pairs(_graph(key, B.BD_LAYOUT_CSR)[0].n, 2, M)
    for R in (40, 100):
        _check(key, B.BD_LAYOUT_CSR, s, t, 41, 5, R, M)  # blocks of 5: a last group of 1 or 2 probes


@pytest.mark.parametrize("key", ["small", "dense"])
def test_split_probes_and_chunk_sizes(key):
    s, t = queries.uniform_pairs(_graph(key, B.BD_LAYOUT_AUTO)[0].n, 2, 8)
    _check(key, B.BD_LAYOUT_AUTO, s, t, 6, 1, 4200, modes=("batched",))
    _check(key, B.BD_LAYOUT_AUTO, s, t, 20, 40, 70, modes=("batched",), chunk_probes=32)
    _check(key, B.BD_LAYOUT_AUTO, s, t, 20, 4, 300, modes=("batched",), chunk_pairs=128, queues=1)


@pytest.mark.parametrize("flags", LAYOUTS)
def test_both_sides_of_the_rule(flags):
    # 1,600 nodes: scored steps 2 R (L + 1) below and above the positions; mixed in one launch
    g, dg = _graph("dense", flags)
    s, t = queries.uniform_pairs(g.n, 12, 21)
    L = np.array([1, 2, 5, 11, 12, 13, 14, 20, 40, 0, 3, 90], dtype=np.int32)
    _check("dense", flags, s, t, L, 2, 60)
    _check("dense", flags, s, t, L, 2, 20)


def test_hub_of_high_degree():
    s, t = np.array([0, 17, 40000], dtype=np.int32), np.array([5, 0, 39999], dtype=np.int32)
    _check("wheel", B.BD_LAYOUT_CSR, s, t, 100, 1, 300)
    _check("wheel", STORAGE, s, t, 100, 1, 300)


def test_served_and_replayed():
    for key in ("small", "dense"):
        g, dg = _graph(key, B.BD_LAYOUT_CSR)
        s, t = queries.uniform_pairs(g.n, 9, 33)
        L = np.array([3, 64, 31, 100, 7, 50, 20, 11, 90], dtype=np.int32)
        pol = B.policy("fixed", B=3, R=90)
        ref = B.bd_query_batch(dg, s, t, 0.1, L, SEED, pol, B.exec_cfg("plain"))
        for _ in range(3):
            got = B.bd_query_batch(dg, s, t, 0.1, L, SEED, pol, B.exec_cfg("batched", use_graph=True))
            assert np.array_equal(got["beta"], ref["beta"])
        srv = B.Server(dg, pol)
        ids = [srv.submit(s, t, 0.1, L, SEED) for _ in range(3)]
        for i in ids:
            assert np.array_equal(srv.wait(i)[0]["beta"], ref["beta"])
        srv.destroy()


@pytest.mark.parametrize("n", [1601, 1634])
@pytest.mark.parametrize("M", [1, 2, 3, 4])
def test_zeros_from_memory(n, M):
    """One or two nodes of a probe have sign 0: read often on a graph of few nodes
    (too many entries for the LDS form), with a last group of fewer probes."""
    key = f"dense{n}"
    GRAPHS.setdefault(key, lambda: graphs.random_connected(n, 0.0375, 6))
    s, t = queries.uniform_pairs(n, 3, M)
    _check(key, B.BD_LAYOUT_CSR, s, t, 61, 5, 70, M)
    _check(key, B.BD_LAYOUT_CSR, s, t, 90, 5, 40, M, modes=("batched",))


@pytest.mark.parametrize("hub", [(1 << 20) - 1, 1 << 20])
def test_hub_of_highest_degree(hub):
    """Degrees are taken from their binary32 reciprocals up to 2^20 - 1."""
    key = f"star{hub}"
    GRAPHS.setdefault(key, lambda: graphs.csr_from_edges(hub + 1, np.zeros(hub, int), np.arange(1, hub + 1)))
    _check(key, B.BD_LAYOUT_CSR, np.array([0], np.int32), np.array([hub], np.int32), 3000, 1, 300, modes=("batched",))
