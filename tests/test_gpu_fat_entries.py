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
