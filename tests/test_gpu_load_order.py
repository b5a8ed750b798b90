"""Loading takes about the same time whatever the order of the ids: the connectivity
check once followed a long path one node at a time where it lay in ascending
order (4e6 nodes: 1.06 s, and 16 ms in any other)."""

import time

import numpy as np
import pytest

from paper_2512_05460_amd import binding as B

pytestmark = pytest.mark.gpu


def cycle(order):
    """CSR of the cycle through the nodes in that order."""
    n = order.size
    ends = np.empty((n, 2), np.int32)
    ends[order, 0], ends[order, 1] = np.roll(order, 1), np.roll(order, -1)
    ends.sort(axis=1)
    return n, 2 * np.arange(n + 1, dtype=np.int64), ends.reshape(-1)


@pytest.mark.parametrize("n", [4_000_000, 2_097_153])
def test_order_of_ids(n):
    took = {}
    rng = np.random.default_rng(1)
    for name, order in (("shuffled", rng.permutation(n)), ("ascending", np.arange(n))):
        g = cycle(order)
        times = []
        for _ in range(3):
            t0 = time.perf_counter()
            dg = B.graph_load_csr(*g, B.BD_LAYOUT_CSR)
            times.append(time.perf_counter() - t0)
            assert dg.info()["bipartite"] == (n % 2 == 0)
            dg.free()
        took[name] = min(times)
    assert took["ascending"] < 5 * took["shuffled"], took
