"""The truncated series' device memory: whole slabs of columns, no more of them than
the pairs fill, and fewer pairs a pass where an allocator gives no more (17 and 33
pairs once took three matrices of as many columns)."""

import ctypes

import numpy as np
import pytest
import torch

from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q,columns", [(17, 17), (33, 33), (48, 48), (64, 64)])
def test_limited_allocator(Q, columns):
    n = 6000
    g = graphs.random_connected(n, 0.001, 2)
    dg = B.graph_load_csr(g.n, g.row_ptr, g.col, B.BD_LAYOUT_CSR)
    s, t = queries.uniform_pairs(n, Q, 3)
    ref = B.bd_truncated_beta(dg, s, t, 30)
    limit, given, most = 3 * 8 * n * columns, {}, [0]

    def alloc(ctx, nbytes, stream):
        if sum(given.values()) + nbytes > limit + 2 ** 20:  # the sums and seeds beside the matrices
            return None
        p = torch.cuda.caching_allocator_alloc(int(nbytes), device=0)
        given[p] = nbytes
        most[0] = max(most[0], nbytes)
        return p

    def free(ctx, ptr, nbytes, stream):
        del given[ptr]
        torch.cuda.caching_allocator_delete(ptr)

    a = B.BdAllocator(None, B._ALLOC_FN(alloc), B._FREE_FN(free))
    B._check(B.lib().bd_set_allocator(ctypes.byref(a)), "bd_set_allocator")
    try:
        got = B.bd_truncated_beta(dg, s, t, 30)
    finally:
        B.use_torch_allocator(True)
    assert not given and most[0] <= 8 * n * -(-Q // 16) * 16 + 256
    # the same sums in slabs of other columns: 30 steps of at most d_max = 20 terms
    assert g.deg.max() <= 20 and np.allclose(got, ref, rtol=31 * 20 * 2.0 ** -52, atol=0)
    dg.free()
