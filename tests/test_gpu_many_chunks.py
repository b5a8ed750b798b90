"""A plain query of more chunks than one launch has work items for (2^32: 4,194,303
work groups of 1,024 threads) runs in several launches."""

import numpy as np
import pytest

from paper_2512_05460_amd import binding as B
from synth import graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags,probes", [(B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE, 114_000)])
def test_plain_query_of_many_chunks(flags, probes):
    g = graphs.workload_graph("ba1k")
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    pol = B.policy("fixed", B=probes, R=2)
    args = (dg, [3], [700], 0.1, 1, graphs.PHILOX_SEED, pol)
    ref = B.bd_query_batch(*args, B.exec_cfg("batched"))
    got, st = B.bd_query_batch(*args, B.exec_cfg("plain", chunk_probes=1), with_stats=True)
    assert got["status"][0] == 0 and st["chunks"] == 37 * probes > 2 ** 32 // 1024 and st["launches"] == 2
    assert np.array_equal(got["beta"], ref["beta"])
    dg.free()
