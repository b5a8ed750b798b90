// Graph loading on the device: the checks of the caller's CSR and the tables
// of the layouts. Everything here streams the adjacency once or twice; on the
// host the same loops took 8 of a load's 12 ms at n = 1e5, 1e6 entries.
#include <algorithm>

#include "pw_internal.hpp"

namespace pw {

// ---------------------------------------------------------------------------
// Checks. A wave takes a row. Bit 0 of *bad: an id outside [0, n); bit 1: a
// self-loop, a row not ascending, or an entry whose mirror is missing (looked
// up by bisection in the neighbour's row). A row's offsets have been checked.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void check_kernel(CsrView g, int deep, uint32_t* bad)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t found = 0;
    for (uint32_t v = blockIdx.x * 4u + (threadIdx.x >> 6); v < g.n; v += gridDim.x * 4u) {
        const int64_t b = g.rp[v], e = g.rp[v + 1];
        for (int64_t i = b + lane; i < e; i += 64) {
            const int32_t u = g.col[i];
            if (u < 0 || (uint32_t)u >= g.n) {
                found |= 1u;
                continue;
            }
            if (!deep) continue;
            if ((uint32_t)u == v || (i > b && g.col[i - 1] >= u)) found |= 2u;
            int64_t lo = g.rp[u], hi = g.rp[u + 1];
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (g.col[mid] < (int32_t)v) lo = mid + 1;
                else hi = mid;
            }
            if (lo >= g.rp[u + 1] || g.col[lo] != (int32_t)v) found |= 2u;
        }
    }
    if (found) atomicOr(bad, found);
}

// ---------------------------------------------------------------------------
// Connectivity and bipartiteness together, on the bipartite double cover: nodes
// (v, side), an edge u-v joining (u, 0) to (v, 1) and (u, 1) to (v, 0). The
// graph is connected when every v has a side in the component of (0, 0), and
// then bipartite when (0, 1) is not in it. Components by union-find: a root is
// hooked under a smaller one by compare-and-swap, so parents only decrease and
// every loop ends; a stale parent read only takes another turn.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t parent_of(uint32_t* p, uint32_t x)
{
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t find_root(uint32_t* p, uint32_t x)
{
    uint32_t q = parent_of(p, x);
    while (q != x) {
        const uint32_t up = parent_of(p, q);
        // halving; atomicMin so that a parent never grows
        if (up != q) atomicMin(p + x, up);
        x = q;
        q = up;
    }
    return x;
}

__device__ __forceinline__ void unite(uint32_t* p, uint32_t a, uint32_t b)
{
    for (;;) {
        a = find_root(p, a);
        b = find_root(p, b);
        if (a == b) return;
        if (a < b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        if (atomicCAS(p + a, a, b) == a) return;  // a > b: a was a root and now hangs under b
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

__global__ __launch_bounds__(256) void cover_unite_kernel(CsrView g, uint32_t* parent)
{
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t v = blockIdx.x * 4u + (threadIdx.x >> 6); v < g.n; v += gridDim.x * 4u) {
        const int64_t b = g.rp[v], e = g.rp[v + 1];
        for (int64_t i = b + lane; i < e; i += 64) {
            const uint32_t u = (uint32_t)g.col[i];
            if (u >= v) continue;  // each edge once
            unite(parent, 2u * v, 2u * u + 1u);
            unite(parent, 2u * v + 1u, 2u * u);
        }
    }
}

// bit 0: not connected; bit 1: (0, 1) is in the component of (0, 0)
__global__ __launch_bounds__(256) void cover_verdict_kernel(uint32_t n, uint32_t* parent, uint32_t* verdict)
{
    const uint32_t r = find_root(parent, 0u);
    uint32_t found = 0;
    for (uint32_t v = blockIdx.x * 256u + threadIdx.x; v < n; v += gridDim.x * 256u) {
        const bool a = find_root(parent, 2u * v) == r, b = find_root(parent, 2u * v + 1u) == r;
        if (!a && !b) found |= 1u;
        if (v == 0 && b) found |= 2u;
    }
    if (found) atomicOr(verdict, found);
}

hipError_t launch_check(const CsrView& g, int deep, uint32_t* bad, hipStream_t st)
{
    hipLaunchKernelGGL(check_kernel, dim3(std::min((g.n + 3u) / 4u, 65536u)), dim3(256), 0, st, g, deep, bad);
    return hipGetLastError();
}

hipError_t launch_components(const CsrView& g, uint32_t* parent, uint32_t* verdict, hipStream_t st)
{
    const dim3 rows(std::min((g.n + 3u) / 4u, 65536u)), nodes(std::min((g.n + 255u) / 256u, 16384u)), block(256);
    hipLaunchKernelGGL(cover_start_kernel, nodes, block, 0, st, g, parent);
    hipLaunchKernelGGL(cover_unite_kernel, rows, block, 0, st, g, parent);
    hipLaunchKernelGGL(cover_verdict_kernel, nodes, block, 0, st, g.n, parent, verdict);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tables. Row i of the result is the caller's row order[i] (i itself without
// an order), its neighbours renamed by `map` (kept without one), as 4-byte or
// as packed 3-byte ids. A wave takes a row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rename_kernel(CsrView g, const uint32_t* order, const uint32_t* map,
                                                     const uint32_t* rp, uint32_t* ids, uint8_t* ids24)
{
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t i = blockIdx.x * 4u + (threadIdx.x >> 6); i < g.n; i += gridDim.x * 4u) {
        const uint32_t v = order ? order[i] : i, to = rp[i], d = rp[i + 1] - to;
        const int32_t* from = g.col + g.rp[v];
        for (uint32_t j = lane; j < d; j += 64u) {
            const uint32_t u = (uint32_t)from[j], x = map ? map[u] : u;
            if (ids) ids[to + j] = x;
            if (ids24) {
                uint8_t* p = ids24 + 3u * (size_t)(to + j);
                p[0] = (uint8_t)x;
                p[1] = (uint8_t)(x >> 8);
                p[2] = (uint8_t)(x >> 16);
            }
        }
    }
}

hipError_t launch_rename(const CsrView& g, const uint32_t* order, const uint32_t* map, const uint32_t* rp, uint32_t* ids,
                         uint8_t* ids24, hipStream_t st)
{
    hipLaunchKernelGGL(rename_kernel, dim3(std::min((g.n + 3u) / 4u, 65536u)), dim3(256), 0, st, g, order, map, rp, ids,
                       ids24);
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

}  // namespace pw
