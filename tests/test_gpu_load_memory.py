"""A graph loads where an allocator has no room for the sign tables beside its own
tables and the copy of its arrays: the general kernels run its queries, and give
the same results."""

import ctypes

import numpy as np
import pytest
import torch

from paper_2512_05460_amd import binding as B
from synth import graphs, queries

pytestmark = pytest.mark.gpu

STORAGE = B.BD_LAYOUT_COMPACT | B.BD_RELABEL_DEGREE | B.BD_PROBE_STORAGE_IDS


@pytest.mark.parametrize("name,flags", [("cl100k", B.BD_LAYOUT_CSR), ("cl100k", STORAGE), ("ba1k", B.BD_LAYOUT_FAT)])
def test_no_room_for_sign_tables(name, flags):
    g = graphs.workload_graph(name)
    s, t = queries.uniform_pairs(g.n, 4, 5)
    args = (s, t, 0.1, [0, 40, 100, 300], graphs.PHILOX_SEED, B.policy("fixed", B=4, R=200))
    full = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
    ref, beta = B.bd_query_batch(full, *args), B.bd_truncated_beta(full, s, t, 50)
    given, peak, room, refused = {}, [0], [1 << 60], [0]

    def alloc(ctx, nbytes, stream):
        if sum(given.values()) + nbytes > room[0]:
            refused[0] += 1
            return None
        p = torch.cuda.caching_allocator_alloc(int(nbytes), device=0)
        given[p] = nbytes
        peak[0] = max(peak[0], sum(given.values()))
        return p

    def free(ctx, ptr, nbytes, stream):
        del given[ptr]
        torch.cuda.caching_allocator_delete(ptr)

    a = B.BdAllocator(None, B._ALLOC_FN(alloc), B._FREE_FN(free))
    B._check(B.lib().bd_set_allocator(ctypes.byref(a)), "bd_set_allocator")
    try:
        B.graph_load_csr(g.n, g.row_ptr, g.col, flags).free()
        assert not given
        room[0] = peak[0] - 256  # the load's largest moment is that of the last sign table
        dg = B.graph_load_csr(g.n, g.row_ptr, g.col, flags)
        room[0] = 1 << 60
        assert refused[0] == 1 and dg.info()["device_bytes"] < full.info()["device_bytes"]
        for mode in ("plain", "batched"):
            got = B.bd_query_batch(dg, *args, B.exec_cfg(mode))
            assert np.all(got["status"] == 0) and np.array_equal(got["beta"], ref["beta"])
        # (another form of the series where the small one needs those tables: 51 steps, d_max < 200)
        assert np.allclose(B.bd_truncated_beta(dg, s, t, 50), beta, rtol=1e-11, atol=0)
        srv = B.Server(dg, B.policy("fixed", B=4, R=200))
        assert np.array_equal(srv.wait(srv.submit(s, t, 0.1, [0, 40, 100, 300], graphs.PHILOX_SEED))[0]["beta"], ref["beta"])
        srv.destroy()
        dg.free()
        assert not given
    finally:
        B.use_torch_allocator(True)
        full.free()
