"""The truncated series is the deterministic reference: a pair gives the same
binary64 value in every call and at every place of a batch. Dense small graphs,
where the order in which rows of many neighbours are worked on differs from run
to run and from work group to work group."""

import numpy as np
import pytest

from oracle import exact as X
from paper_2512_05460_amd import binding as B
from synth import graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p", [(1000, 0.03), (700, 0.04), (1500, 0.02)])
def test_the_same_every_time(n, p):
    g = graphs.random_connected(n, p, 8)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR)
    assert np.sum(np.diff(g.row_ptr) > 16) > 500
    s, t = np.full(48, 3, np.int32), np.full(48, n - 5, np.int32)
    ref = B.bd_truncated_beta(dg, s, t, 300)
    # both sides round a sum of at most d_max < 70 terms per entry and step and P has norm 1
    assert ref[0] == pytest.approx(X.beta_truncated(g, 3, n - 5, 300), rel=300 * 70 * 2.0 ** -53)
    assert np.all(ref == ref[0])
    for _ in range(6):
        assert np.array_equal(B.bd_truncated_beta(dg, s, t, 300), ref)
    dg.free()
