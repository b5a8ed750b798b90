"""Two servers on one loaded graph, their requests submitted in turn and collected
in another order: every result equals the batched one bit for bit, in every
pass. One server's queries run on the general kernels (few replicas, requests
of 1 to 64 pairs), the other's on the sign tables; slots are taken over by
later requests."""

import numpy as np
import pytest

from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu

SEED = graphs.PHILOX_SEED


@pytest.mark.parametrize("flags", [B.BD_LAYOUT_FAT, B.BD_LAYOUT_CSR])
def test_two_servers(flags):
    g = graphs.random_connected(5000, 0.002, 9)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    sizes = [1, 8, 64, 2, 16, 1, 32, 4]
    s, t = queries.uniform_pairs(g.n, sum(sizes), 12)
    at = np.concatenate([[0], np.cumsum(sizes)])
    runs = []
    for few, L in ((True, 120), (False, 60)):
        pol = B.policy("fixed", B=8, R=3 if few else 100)
        ref = B.bd_query_batch(dg, s, t, 0.1, L, SEED + few, pol, B.exec_cfg("batched"))
        assert np.all(ref["status"] == 0)
        runs.append((B.Server(dg, pol, max_queries=70), L, SEED + few, ref["beta"]))
    for rep in range(3):
        ids = [[srv.submit(s[a:b], t[a:b], 0.1, L, seed, uid=np.arange(a, b)) for srv, L, seed, _ in runs]
               for a, b in zip(at[:-1], at[1:])]
        for k in reversed(range(len(sizes))):
            for (srv, _, _, ref), i in zip(runs, ids[k]):
                got = srv.wait(i)[0]["beta"]
                assert np.array_equal(got, ref[at[k]:at[k + 1]]), (rep, k)
    for srv, *_ in runs:
        srv.destroy()
    dg.free()
