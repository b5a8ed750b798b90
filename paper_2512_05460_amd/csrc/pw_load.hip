// Graph loading on the device: the checks of the caller's CSR and the tables
// of the layouts. Everything here streams the adjacency once or twice; on the
// host the same loops took 8 of a load's 12 ms at n = 1e5, 1e6 entries.
#include <algorithm>

#include "pw_internal.hpp"

namespace pw {

// The row of entry i, of n rows with offsets rp: rp[v] <= i < rp[v + 1]. The
// kernels over entries give every thread one, so that a long row holds nobody up
// (with a wave a row, a star of 60,000 leaves loaded in 1.39 ms, now in 0.58, and
// check_kernel took 100 us at 1e6 entries, now 44); a wave's bisections share
// their lines nearly to the end.
template <typename T>
__device__ __forceinline__ uint32_t row_of(const T* rp, uint32_t n, T i)
{
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1u) {
        const uint32_t mid = lo + (hi - lo) / 2u;
        if (rp[mid] <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Checks. Bit 0 of *bad: an id outside [0, n); bit 1: a self-loop, a row not
// ascending, or an entry whose mirror is missing (looked up by bisection in the
// neighbour's row). The offsets have been checked.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void check_kernel(CsrView g, int64_t nnz, int deep, uint32_t* bad)
{
    uint32_t found = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * 256) {
        const int32_t u = g.col[i];
        if (u < 0 || (uint32_t)u >= g.n) {
            found |= 1u;
            continue;
        }
        if (!deep) continue;
        const uint32_t v = row_of(g.rp, g.n, i);
        if ((uint32_t)u == v || (i > g.rp[v] && g.col[i - 1] >= u)) found |= 2u;
        int64_t a = g.rp[u], e = g.rp[u + 1];
        const int64_t end = e;
        while (a < e) {
            const int64_t mid = (a + e) >> 1;
            if (g.col[mid] < (int32_t)v) a = mid + 1;
            else e = mid;
        }
        if (a >= end || g.col[a] != (int32_t)v) found |= 2u;
    }
    if (found) atomicOr(bad, found);
}

// ---------------------------------------------------------------------------
// Connectivity and bipartiteness together, on the bipartite double cover: nodes
// (v, side), an edge u-v joining (u, 0) to (v, 1) and (u, 1) to (v, 0). The
// graph is connected when every v has a side in the component of (0, 0), and
// then bipartite when (0, 1) is not in it. Components by union-find: only the
// larger end climbs, and a root is hooked under a smaller node by
// compare-and-swap, so parents are always smaller and every loop ends. A parent
// read may be an old one: it is an ancestor still, and what looks like a root
// but is none is told by the compare-and-swap. Atomics on one line go one after
// another (40 ns each): a climb therefore writes nothing before its eighth step,
// and each kernel starts from copies that hang right under their roots. At
// n = 1e5 and 1e6 entries the seven launches take 0.19 ms, 0.15 of them
// cover_last_kernel's compare-and-swaps at the large components' roots; with
// every edge united at once, each climb halving its path, they took 1.4 ms.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t parent_of(const uint32_t* p, uint32_t x)
{
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void hang(uint32_t* p, uint32_t x, uint32_t ancestor)
{
    __hip_atomic_store(p + x, ancestor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void unite(uint32_t* p, uint32_t a, uint32_t b)
{
    for (uint32_t steps = 0; a != b; ++steps) {
        if (a < b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        uint32_t up = parent_of(p, a);
        if (up == a) {
            up = atomicCAS(p + a, a, b);
            if (up == a) return;  // a was a root and now hangs under b
        } else if (steps >= 8) {  // a long climb halves its path; a is no root, so nobody else needs its entry
            const uint32_t next = parent_of(p, up);
            if (next != up) hang(p, a, up = next);
        }
        a = up;
    }
}

// The start: every copy hangs under its row's first neighbour's other copy where
// that is smaller, which joins most of the graph without contention.
__global__ __launch_bounds__(256) void cover_start_kernel(CsrView g, uint32_t* parent)
{
    for (uint32_t v = blockIdx.x * 256u + threadIdx.x; v < g.n; v += gridDim.x * 256u) {
        const uint32_t u = (uint32_t)g.col[g.rp[v]];
        parent[2u * v] = u < v ? 2u * u + 1u : 2u * v;
        parent[2u * v + 1u] = u < v ? 2u * u : 2u * v + 1u;
    }
}

// Every copy right under its root. Each step is written at once, so that the
// others' steps get longer by it: of a path of n nodes that are worked on together
// each takes about log n. A thread takes one copy, so that copies are begun in
// ascending order and what lies below the ones at work hangs under its root
// already: where threads took a second copy when done with the first, a cycle of
// 4e6 nodes in order, whose later copies then came before the middle ones, loaded
// in 1,056 ms, now in 16.
__global__ __launch_bounds__(256) void cover_flatten_kernel(uint32_t copies, uint32_t* parent)
{
    const uint32_t x = blockIdx.x * 256u + threadIdx.x;
    if (x >= copies) return;
    uint32_t up = __hip_atomic_load(parent + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        const uint32_t next = __hip_atomic_load(parent + up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (next == up) break;
        hang(parent, x, up = next);
    }
}

// One more edge of every node: its row's last. With the first ones that leaves
// one or two components but for a remainder.
__global__ __launch_bounds__(256) void cover_last_kernel(CsrView g, uint32_t* parent)
{
    for (uint32_t v = blockIdx.x * 256u + threadIdx.x; v < g.n; v += gridDim.x * 256u) {
        const uint32_t u = (uint32_t)g.col[g.rp[v + 1] - 1];
        unite(parent, 2u * v, 2u * u + 1u);
        unite(parent, 2u * v + 1u, 2u * u);
    }
}

// Every edge, once: the two ends of nearly all hang under one root already.
__global__ __launch_bounds__(256) void cover_unite_kernel(CsrView g, int64_t nnz, uint32_t* parent)
{
    const uint2* above = reinterpret_cast<const uint2*>(parent);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * 256) {
        const uint32_t v = row_of(g.rp, g.n, i), u = (uint32_t)g.col[i];
        if (u >= v) continue;
        const uint2 pv = above[v], pu = above[u];
        if (pu.y != pv.x) unite(parent, 2u * v, 2u * u + 1u);
        if (pu.x != pv.y) unite(parent, 2u * v + 1u, 2u * u);
    }
}

// bit 0: not connected; bit 1: (0, 1) is in the component of (0, 0). Parents are
// roots here, and (0, 0), the smallest copy, is its component's.
__global__ __launch_bounds__(256) void cover_verdict_kernel(uint32_t n, const uint2* parent, uint32_t* verdict)
{
    uint32_t found = 0;
    for (uint32_t v = blockIdx.x * 256u + threadIdx.x; v < n; v += gridDim.x * 256u) {
        const uint2 p = parent[v];
        if (p.x != 0u && p.y != 0u) found |= 1u;
        if (v == 0 && p.y == 0u) found |= 2u;
    }
    if (found) atomicOr(verdict, found);
}

static dim3 entry_blocks(int64_t nnz) { return dim3((uint32_t)std::min<int64_t>((nnz + 255) / 256, 65536)); }

hipError_t launch_check(const CsrView& g, int64_t nnz, int deep, uint32_t* bad, hipStream_t st)
{
    hipLaunchKernelGGL(check_kernel, entry_blocks(nnz), dim3(256), 0, st, g, nnz, deep, bad);
    return hipGetLastError();
}

hipError_t launch_components(const CsrView& g, int64_t nnz, uint32_t* parent, uint32_t* verdict, hipStream_t st)
{
    const dim3 nodes(std::min((g.n + 255u) / 256u, 16384u)), block(256);
    const dim3 copies((2u * g.n + 255u) / 256u);
    hipLaunchKernelGGL(cover_start_kernel, nodes, block, 0, st, g, parent);
    hipLaunchKernelGGL(cover_flatten_kernel, copies, block, 0, st, 2u * g.n, parent);
    hipLaunchKernelGGL(cover_last_kernel, nodes, block, 0, st, g, parent);
    hipLaunchKernelGGL(cover_flatten_kernel, copies, block, 0, st, 2u * g.n, parent);
    hipLaunchKernelGGL(cover_unite_kernel, entry_blocks(nnz), block, 0, st, g, nnz, parent);
    hipLaunchKernelGGL(cover_flatten_kernel, copies, block, 0, st, 2u * g.n, parent);
    hipLaunchKernelGGL(cover_verdict_kernel, nodes, block, 0, st, g.n, reinterpret_cast<const uint2*>(parent), verdict);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tables. Row i of the result is the caller's row order[i] (i itself without
// an order), its neighbours renamed by `map` (kept without one), as 4-byte or
// as packed 3-byte ids.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rename_kernel(CsrView g, uint32_t nnz, const uint32_t* order, const uint32_t* map,
                                                     const uint32_t* rp, uint32_t* ids, uint8_t* ids24)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * 256) {
        int64_t from = i;
        if (order) {
            const uint32_t row = row_of(rp, g.n, (uint32_t)i);
            from = g.rp[order[row]] + (int64_t)((uint32_t)i - rp[row]);
        }
        const uint32_t u = (uint32_t)g.col[from], x = map ? map[u] : u;
        if (ids) ids[i] = x;
        if (ids24) {
            uint8_t* p = ids24 + 3 * i;
            p[0] = (uint8_t)x;
            p[1] = (uint8_t)(x >> 8);
            p[2] = (uint8_t)(x >> 16);
        }
    }
}

hipError_t launch_rename(const CsrView& g, uint32_t nnz, const uint32_t* order, const uint32_t* map, const uint32_t* rp,
                         uint32_t* ids, uint8_t* ids24, hipStream_t st)
{
    hipLaunchKernelGGL(rename_kernel, entry_blocks(nnz), dim3(256), 0, st, g, nnz, order, map, rp, ids, ids24);
    return hipGetLastError();
}

// Node entries {row offset, degree, bits of 1.0f/degree, original id}, or {row
// offset, original id} with the closing entry {nnz, 0}.
__global__ __launch_bounds__(256) void nodes_kernel(uint32_t n, const uint32_t* order, const uint32_t* rp, uint4* node,
                                                    uint2* node8)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i <= n; i += gridDim.x * 256u) {
        const uint32_t off = rp[i];
        if (i == n) {
            if (node8) node8[n] = make_uint2(off, 0u);
            continue;
        }
        const uint32_t v = order ? order[i] : i, d = rp[i + 1] - off;
        if (node) node[i] = make_uint4(off, d, __float_as_uint(__fdiv_rn(1.0f, (float)d)), v);
        if (node8) node8[i] = make_uint2(off, v);
    }
}

hipError_t launch_nodes(uint32_t n, const uint32_t* order, const uint32_t* rp, uint4* node, uint2* node8, hipStream_t st)
{
    hipLaunchKernelGGL(nodes_kernel, dim3(std::min(n / 256u + 1u, 16384u)), dim3(256), 0, st, n, order, rp, node, node8);
    return hipGetLastError();
}

// Positions and probe ids of the sign-table kernels (SignTables::pid), from the runs
// of equal degree: node i of the descending order has position pos + (i - first) of
// its run. at: by caller id; rank: by i, or null. pid: of each word of 32 positions
// the ids that probes are evaluated on, of 64 words 4 ids at a time; positions of a
// word behind a run's last node repeat its id. (Four loops over the nodes on the
// host, and two more copies up, took 5 of a load's 11.5 ms at n = 1e6.)
__global__ __launch_bounds__(256) void sign_positions_kernel(uint32_t n, const uint32_t* order, const SignRun* runs,
                                                             uint32_t nruns, int ranked, uint32_t* at, uint32_t* rank,
                                                             uint32_t* pid)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        uint32_t lo = 0, hi = nruns;
        while (hi - lo > 1u) {
            const uint32_t mid = lo + (hi - lo) / 2u;
            if (runs[mid].first <= i) lo = mid;
            else hi = mid;
        }
        const SignRun r = runs[lo], next = runs[lo + 1];
        const uint32_t v = order[i], id = ranked ? i : v, x = r.pos + (i - r.first);
        at[v] = x;
        if (rank) rank[i] = x;
        const uint32_t w = r.word + (x / 32u - r.pos / 32u);
        auto put = [&](uint32_t y) { pid[(w / 64u) * 2048u + (y / 4u) * 256u + (w % 64u) * 4u + y % 4u] = id; };
        put(x % 32u);
        if (i + 1u == next.first)
            for (uint32_t y = x + 1u; y % 32u != 0u && y < next.pos; ++y) put(y % 32u);
    }
}

hipError_t launch_sign_positions(uint32_t n, const uint32_t* order, const SignRun* runs, uint32_t nruns, int ranked,
                                 uint32_t* at, uint32_t* rank, uint32_t* pid, hipStream_t st)
{
    hipLaunchKernelGGL(sign_positions_kernel, dim3(std::min((n + 255u) / 256u, 16384u)), dim3(256), 0, st, n, order, runs,
                       nruns, ranked, at, rank, pid);
    return hipGetLastError();
}

}  // namespace pw
