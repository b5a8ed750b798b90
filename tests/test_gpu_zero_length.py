"""Batches whose queries all have L = 0 and replicas enough for the sign tables,
on graphs where the first launch shapes are empty: the adjacency in LDS, and
walk sharing from memory. Every way to run a batch, against the oracle, bit
for bit."""

import numpy as np
import pytest

from oracle import estimator as E
from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu

SEED = graphs.PHILOX_SEED


@pytest.mark.parametrize("n,p,R,M", [(6000, 0.001, 4096, 1), (5000, 0.0012, 2600, 1), (2500, 0.014, 4000, 2),
                                     (2500, 0.014, 4000, 4)])
def test_all_of_length_zero(n, p, R, M):
    g = graphs.random_connected(n, p, 4)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR)
    s, t = queries.uniform_pairs(n, 3, R)
    pol, uid = B.policy("fixed", B=4, R=R, share=M), np.arange(3) + 2
    for L in (0, [0, 0, 1]):
        L = np.broadcast_to(np.array(L, np.int32), 3)
        ref = E.estimate(g, s, t, L, [(4, 37, 148, R)] * 3, SEED, uid=uid, threads=8, share=M)
        for run, ex in ((B.bd_query_batch, B.exec_cfg("plain")), (B.bd_query_batch, B.exec_cfg("batched")),
                        (B.bd_query_batch, B.exec_cfg("batched", use_graph=True)),
                        (B.bd_query_batch_noalloc, B.exec_cfg("batched"))):
            got = run(dg, s, t, 0.1, L, SEED, pol, ex, uid=uid)
            assert np.all(got["status"] == 0) and np.array_equal(got["beta"], ref), (run.__name__, ex.mode, ex.use_graph, L)
    dg.free()
