// Walk kernels that score against sign tables in LDS.
//
// A probe's sign z^(k)(x) is a fixed function of the node. A chunk scores each
// of its probes 2 R (L + 1) times, and where that is more often than the graph
// has nodes it is cheaper to evaluate the Feistel permutation and the hash once
// per node into a table in LDS and let the walks look the sign up: 29
// vector instructions per walk step, the tables' building included, instead of
// 118. The tables are indexed by the
// node's position in the kernels' own tables, so the walks need neither the
// caller's id nor a row table from memory whatever layout the graph was loaded
// in. Two forms:
//
//   * Small graphs (kLds): row offset and degree of every node (4 bytes) and the
//     whole adjacency (2 bytes an entry) are staged in LDS, and a table holds
//     z / d as binary32. A step is three LDS reads.
//   * Larger ones: nodes are stored in descending degree, each run of equal
//     degree padded to whole blocks of 2^shift positions, so a block has one
//     degree d and a node x of it has row offset base + x d. One LDS read of
//     the block's entry {base, bits of 1.0f/d} resolves a node: no search, no
//     second dependent read from memory. A step reads one
//     neighbour position, 3 bytes, from memory (an L2 hit up to about 1.3
//     million adjacency entries); a table holds a bit a node, the sign. z = 0 has
//     one or two nodes a probe at most, which the walks compare with.
//
// The walks, their random streams, the order of the binary32 sums and all
// results are those of the other kernels.
//
// Bounds, and times before (the general kernels) and now: small graphs by LDS
// reads and Philox (32 queries, n = 1,000: 34.0 -> 5.24 ms); one probe a walk by
// the L2s' requests, 2.7e11 a second (256 probes in 37 blocks, L = 1,000, n =
// 1e5: 71.4 -> 68.0 ms of 66; 17 queries on 3-byte ids without hub tables: 60.4
// -> 37.6 of 35); four probes a walk by those and the table building about alike
// (n = 1e5: 24.3 -> 9.5 ms of 8.5). Two bits a node and 16-byte block entries
// took 13.7 ms there: a CU held one work group, and built or walked.
#include "pw_chunk.hpp"
#include "pw_device.hpp"
#include "pw_internal.hpp"

namespace pw {

// Dynamic LDS of a work group, in this order.
struct SignLds {
    uint4* blk;                 // nblk block entries of 8 bytes; kLds: rows, then the adjacency
    unsigned long long* acc;    // T x {S1, S2}
    uint32_t* zero;             // T x two positions with z = 0, ~0 for none (not with kLds)
    uint32_t* tab;              // T tables of tabw words (kMaxG + 2 doubles at least)
};

template <int kLds>
struct SignNode;

template <>
struct SignNode<0> {
    uint32_t x, off, deg;
    float inv;
};

// x4: 4 times the node's id, the byte offset of its row and table entries
template <>
struct SignNode<1> {
    uint32_t x4, row;
};

template <int kLds>
__device__ __forceinline__ SignNode<kLds> sign_node(const SignTables& S, const SignLds& M, uint32_t x)
{
    if constexpr (kLds) {
        return SignNode<1>{x, *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(M.blk) + x)};
    } else {
        const uint2 e = reinterpret_cast<const uint2*>(M.blk)[x >> S.shift];
        const float inv = __uint_as_float(e.y);
        // d < 2^20: v_rcp_f32's 1 ulp and inv's half leave 1/inv less than 1/4 away from it
        const uint32_t d = (uint32_t)(__builtin_amdgcn_rcpf(inv) + 0.5f);
        return SignNode<0>{x, umul24(x, d) + e.x, d, inv};
    }
}

// Neighbour floor(u d / 2^32) of a node (4 times its id with kLds).
template <int kLds>
__device__ __forceinline__ uint32_t sign_next(const SignTables& S, const SignLds& M, const SignNode<kLds>& w, uint32_t u)
{
    if constexpr (kLds) {
        const uint32_t at = ((w.row & 0xFFFFu) + __umulhi(u, w.row >> 16)) << 1;
        return *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(M.blk) + S.nblk * 4u + at);
    } else {
        uint32_t v;  // 4 bytes from byte 3 pos on; the table has 8 bytes of padding
        __builtin_memcpy(&v, reinterpret_cast<const char*>(S.ids) + (w.off + __umulhi(u, w.deg)) * 3u, 4);
        return v & 0xFFFFFFu;
    }
}

// Fills the tables of the phase's gn groups from gi on, whose kn probes start at
// kA. Each wave takes 64 words of one probe (kLds), or of one group, whose words
// hold its kShare probes' bits of a position side by side; the keys are
// wave-uniform. A bit tells a sign and the first position's are on top; a
// probe's one or two zeros are kept as positions.
template <int kLds, int kShare>
__device__ __forceinline__ void sign_build(const SignTables& S, const SignLds& M, const Domain& dom, const QueryDesc& d,
                                           uint32_t gi, uint32_t gn, uint32_t M_, uint32_t gpb, uint32_t kA, uint32_t kn)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
    uint32_t cur = 0xFFFFFFFFu;
    if constexpr (kLds) {
        const uint32_t segs = (S.tabw + 63u) >> 6;
        Probe pr{};
        for (uint32_t u = wave; u < kn * segs; u += nw) {
            const uint32_t j = u / segs;
            if (j != cur) {
                pr = make_probe(d.seed_lo, d.seed_hi, d.uid, kA + j, dom.n);
                cur = j;
            }
            const uint32_t w = (u - j * segs) * 64u + lane;
            if (w >= S.tabw) continue;
            uint32_t y;
            const uint32_t deg = reinterpret_cast<const uint32_t*>(M.blk)[w] >> 16;
            M.tab[j * S.tabw + w] =
                __float_as_uint(__fmul_rn((float)probe_value(w, pr, dom, &y), __fdiv_rn(1.0f, (float)deg)));
        }
    } else {
        constexpr uint32_t kQuads = 8 / kShare;  // a word's positions, four at a time
        const uint32_t segs = (S.words + 63u) >> 6, units = segs * kShare;
        Probe pr[kShare];
        uint32_t m = 0;
        for (uint32_t u = wave; u < gn * units; u += nw) {
            const uint32_t gg = u / units, r = u - gg * units, seg = r / kShare, part = r % kShare;
            if (gg != cur) {
                uint32_t kf;
                group_probes(gi + gg, d.B, M_, gpb, &kf, &m);
#pragma unroll
                for (int j = 0; j < kShare; ++j)
                    if (kShare == 1 || (uint32_t)j < m) pr[j] = make_probe(d.seed_lo, d.seed_hi, d.uid, kf + j, dom.n);
                cur = gg;
            }
            const uint32_t w = seg * 64u + lane;
            if (w >= S.words) continue;
            const uint32_t at = S.pid[2048u * segs + w];  // 32 positions from 32 at on
            const uint4* ids = reinterpret_cast<const uint4*>(S.pid) + (size_t)seg * 512u + part * kQuads * 64u + lane;
            uint32_t word = 0;
#pragma unroll 1
            for (uint32_t i = 0; i < kQuads; ++i) {
                const uint4 v = ids[64u * i];
                uint32_t bits = 0;
#pragma unroll
                for (int j = 0; j < kShare; ++j) {
                    if (kShare != 1 && (uint32_t)j >= m) break;
                    const Probe& q = pr[j];
                    // four permutations at once; the few values that land past n are walked on
                    uint32_t y[4] = {feistel_once(v.x, q, dom), feistel_once(v.y, q, dom), feistel_once(v.z, q, dom),
                                     feistel_once(v.w, q, dom)};
                    while (max(max(y[0], y[1]), max(y[2], y[3])) >= dom.n) {
#pragma unroll
                        for (int h = 0; h < 4; ++h)
                            if (y[h] >= dom.n) y[h] = feistel_once(y[h], q, dom);
                    }
#pragma unroll
                    for (int h = 0; h < 4; ++h)
                        bits |= (hash_bit(q, y[h] >> 1) ^ (y[h] & 1u)) << (kShare * (3 - h) + kShare - 1 - j);
                    if (max(max(y[0], y[1]), max(y[2], y[3])) >= q.zlo) {
                        // padding repeats the id before it, whose position is the lower one
                        const uint32_t x = 32u * at + 4u * (part * kQuads + i);
                        uint32_t* z = M.zero + 2u * (gg * kShare + j);
#pragma unroll
                        for (int h = 0; h < 4; ++h)
                            if (y[h] >= q.zlo) atomicMin(z + (y[h] - q.zlo), x + h);
                    }
                }
                word = (word << (4 * kShare)) | bits;
            }
            M.tab[(gg * S.tabw + at) * kShare + part] = word;
        }
    }
}

// The positions of a group's zeros, two a probe.
template <int kLds, int kUniform, int kShare>
struct SignZeros {
    uint32_t z[kLds ? 1 : 2 * kShare];
    __device__ __forceinline__ void read(const uint32_t* zero)
    {
        if constexpr (!kLds) {
#pragma unroll
            for (int i = 0; i < 2 * kShare; ++i) z[i] = kUniform ? __builtin_amdgcn_readfirstlane(zero[i]) : zero[i];
        }
    }
};

// z_j of node w from its word, times 1 / d: +0 for z = 0, which leaves a sum as it
// is (they are never -0).
__device__ __forceinline__ float sign_term(const SignNode<0>& w, uint32_t word, int j, const uint32_t* z)
{
    const uint32_t v = ((word << j) & 0x80000000u) | __float_as_uint(w.inv);
    return w.x == z[2 * j] || w.x == z[2 * j + 1] ? 0.0f : __uint_as_float(v);
}

// Scores both walks' nodes against the m probes of a group whose tables start at tab.
template <int kLds, int kUniform, int kShare>
__device__ __forceinline__ void sign_score(const SignTables& S, const uint32_t* tab,
                                           const SignZeros<kLds, kUniform, kShare>& Z, uint32_t m, const SignNode<kLds>& s,
                                           const SignNode<kLds>& t, float* a, float* b)
{
    if constexpr (kLds) {
#pragma unroll
        for (int j = 0; j < kShare; ++j) {
            if (kShare == 1 || (uint32_t)j < m) {
                const char* row = reinterpret_cast<const char*>(tab + j * S.tabw);
                a[j] = __fadd_rn(a[j], *reinterpret_cast<const float*>(row + s.x4));
                b[j] = __fadd_rn(b[j], *reinterpret_cast<const float*>(row + t.x4));
            }
        }
    } else {
        const uint32_t bs = s.x * kShare, bt = t.x * kShare;
        const uint32_t ws = tab[bs >> 5] << (bs & 31u), wt = tab[bt >> 5] << (bt & 31u);
#pragma unroll
        for (int j = 0; j < kShare; ++j) {
            if (kShare == 1 || (uint32_t)j < m) {
                a[j] = __fadd_rn(a[j], sign_term(s, ws, j, Z.z));
                b[j] = __fadd_rn(b[j], sign_term(t, wt, j, Z.z));
            }
        }
    }
}

// U_p of replica p for the m probes of a group, whose tables start at tab (the
// streams are keyed by kw, the group's first probe). The two neighbour reads of
// a step are issued before the nodes just left are scored.
template <int kLds, int kUniform, int kShare>
__device__ __forceinline__ void sign_pair(const SignTables& S, const SignLds& M, const uint32_t* tab,
                                          const SignZeros<kLds, kUniform, kShare>& Z, uint32_t m,
                                          SignNode<kLds> s, SignNode<kLds> t, int L, uint32_t p, uint32_t kw, uint32_t uid,
                                          uint32_t slo, uint32_t shi, float* U)
{
    float a[kShare], b[kShare];
#pragma unroll
    for (int j = 0; j < kShare; ++j) a[j] = b[j] = 0.0f;
    auto score = [&]() { sign_score<kLds, kUniform, kShare>(S, tab, Z, m, s, t, a, b); };
    auto advance2 = [&](uint32_t us, uint32_t ut) {
        const uint32_t xs = sign_next<kLds>(S, M, s, us);
        const uint32_t xt = sign_next<kLds>(S, M, t, ut);
        score();
        s = sign_node<kLds>(S, M, xs);
        t = sign_node<kLds>(S, M, xt);
    };
    const uint32_t cs = uid << 1, ct = (uid << 1) | 1u;
    const int full = L >> 2;
    for (int blk = 0; blk < full; ++blk) {
        const U4 rs = philox10_walk((uint32_t)blk, p, kw, cs, slo, shi);
        const U4 rt = philox10_walk((uint32_t)blk, p, kw, ct, slo, shi);
        advance2(rs.x, rt.x);
        advance2(rs.y, rt.y);
        advance2(rs.z, rt.z);
        advance2(rs.w, rt.w);
    }
    const int rem = L & 3;
    if (rem) {
        const U4 rs = philox10_walk((uint32_t)full, p, kw, cs, slo, shi);
        const U4 rt = philox10_walk((uint32_t)full, p, kw, ct, slo, shi);
        advance2(rs.x, rt.x);
        if (rem > 1) advance2(rs.y, rt.y);
        if (rem > 2) advance2(rs.z, rt.z);
    }
    score();
#pragma unroll
    for (int j = 0; j < kShare; ++j) U[j] = __fsub_rn(a[j], b[j]);
}

template <int kLds, int kUniform, int kShare>
__device__ __forceinline__ void sign_chunk(const WalkArgs& A, const SignLds& M, uint32_t ci, uint32_t* flag)
{
    double* ys = reinterpret_cast<double*>(M.tab);  // block means, once the tables have been used
    const Chunk c = A.chunks[ci];
    const QueryDesc d = A.qd[c.q];
    const SignTables& S = A.signs;
    Domain dom;
    dom.n = A.g.dom.n;
    dom.rb = A.g.dom.rb;
    dom.mask = A.g.dom.mask;
    dom.rsh = A.g.dom.rsh;
    dom.A = A.g.dom.A;
    dom.A8 = A.g.dom.A8;
    const uint32_t M_ = kShare == 1 ? 1u : d.share;
    const uint32_t gpb = (d.B + M_ - 1) / M_;
    const uint32_t slots = kLds ? M_ : (uint32_t)kShare;  // tables of a group
    const uint32_t per_phase = max(1u, S.T / slots);
    const uint32_t tid = threadIdx.x, kT = blockDim.x;
    const SignNode<kLds> s0 = sign_node<kLds>(S, M, d.ss), t0 = sign_node<kLds>(S, M, d.st);
    // phases of as many groups as there are tables
    for (uint32_t g = 0; g < c.gc; g += per_phase) {
        const uint32_t gn = min(per_phase, c.gc - g);
        uint32_t kA, kl, sz;
        group_probes(c.g0 + g, d.B, M_, gpb, &kA, &sz);
        group_probes(c.g0 + g + gn - 1u, d.B, M_, gpb, &kl, &sz);
        const uint32_t kn = kl + sz - kA;
        for (uint32_t j = tid; j < kn * 4u; j += kT) M.acc[j] = 0ull;
        if constexpr (!kLds) {
            for (uint32_t j = tid; j < gn * kShare * 2u; j += kT) M.zero[j] = 0xFFFFFFFFu;
            __syncthreads();
        }
        sign_build<kLds, kShare>(S, M, dom, d, c.g0 + g, gn, M_, gpb, kA, kn);
        __syncthreads();
        if constexpr (kUniform) {
            // each wave takes 64 consecutive replicas of one group
            const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            const uint32_t lane = tid & 63u;
            const uint32_t nb = (c.pc + 63u) >> 6;
            const uint32_t pend = c.p0 + c.pc;
            for (uint32_t u = wave; u < gn * nb; u += kT >> 6) {
                const uint32_t gg = u / nb;
                const uint32_t p = c.p0 + (u - gg * nb) * 64u + lane;
                uint32_t kf, m;
                group_probes(c.g0 + g + gg, d.B, M_, gpb, &kf, &m);
                const uint32_t slot = kLds ? kf - kA : gg * kShare;
                SignZeros<kLds, kUniform, kShare> Z;
                Z.read(M.zero + 2u * slot);
                if (p < pend) {
                    float U[kShare];
                    sign_pair<kLds, kUniform, kShare>(S, M, M.tab + slot * S.tabw, Z, m, s0, t0, d.L, p, kf, d.uid, d.seed_lo,
                                            d.seed_hi, U);
#pragma unroll
                    for (int j = 0; j < kShare; ++j) {
                        if (kShare == 1 || (uint32_t)j < m) {
                            unsigned long long* a4 = M.acc + 4 * (kf + j - kA);
                            lds_add_i128(a4, fix54(U[j]));
                            lds_add_i128(a4 + 2, (i128)sqfix64(U[j]));
                        }
                    }
                }
            }
        } else {
            // lanes over the phase's (group, replica) pairs
            const uint64_t total = (uint64_t)gn * c.pc;
            for (uint64_t w = tid; w < total; w += kT) {
                const uint32_t gg = (uint32_t)(w / c.pc);
                const uint32_t p = c.p0 + (uint32_t)(w - (uint64_t)gg * c.pc);
                uint32_t kf, m;
                group_probes(c.g0 + g + gg, d.B, M_, gpb, &kf, &m);
                const uint32_t slot = kLds ? kf - kA : gg * kShare;
                SignZeros<kLds, kUniform, kShare> Z;
                Z.read(M.zero + 2u * slot);
                float U[kShare];
                sign_pair<kLds, kUniform, kShare>(S, M, M.tab + slot * S.tabw, Z, m, s0, t0, d.L, p, kf, d.uid, d.seed_lo,
                                        d.seed_hi, U);
#pragma unroll
                for (int j = 0; j < kShare; ++j) {
                    if (kShare == 1 || (uint32_t)j < m) {
                        unsigned long long* a4 = M.acc + 4 * (kf + j - kA);
                        lds_add_i128(a4, fix54(U[j]));
                        lds_add_i128(a4 + 2, (i128)sqfix64(U[j]));
                    }
                }
            }
        }
        __syncthreads();
        if (c.pc < d.R) finish_parts(A, d, kA, kn, c.pc, M.acc, ys, flag);
        else finish_probes(A, d, kA, kn, M.acc, ys, flag, kT);
    }
}

template <int kLds, int kUniform, int kShare>
__global__ __launch_bounds__(1024, kShare == 1 ? 8 : 4) void sign_kernel(WalkArgs A)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t next;
    __shared__ uint32_t qstate[2];
    const SignTables& S = A.signs;
    SignLds M;
    // staged: the block entries, or the rows and the adjacency (whole 16 bytes)
    const uint32_t staged = kLds ? (S.nblk + S.idw) / 4u : S.nblk / 2u;
    M.blk = reinterpret_cast<uint4*>(lds);
    M.acc = reinterpret_cast<unsigned long long*>(M.blk + staged);
    M.zero = reinterpret_cast<uint32_t*>(M.acc + 4u * S.T);
    M.tab = M.zero + 2u * S.T;
    for (uint32_t i = threadIdx.x; i < staged; i += blockDim.x) M.blk[i] = S.blk[i];
    if (!A.persistent) {
        if (threadIdx.x == 0) next = abort_raised(A) ? 1u : 0u;
        __syncthreads();
        if (blockIdx.x < A.nchunks && next == 0u) sign_chunk<kLds, kUniform, kShare>(A, M, blockIdx.x, &next);
        return;
    }
    if (threadIdx.x == 0) first_queue(A, qstate);
    for (;;) {
        if (threadIdx.x == 0) next = claim_chunk(A, qstate);
        __syncthreads();
        const uint32_t ci = next;
        __syncthreads();
        if (ci >= A.nchunks) break;
        sign_chunk<kLds, kUniform, kShare>(A, M, ci, &next);
    }
}

typedef void (*SignKernel)(WalkArgs);

template <int kLds>
static SignKernel sign_fn_l(int uniform, int share)
{
    if (share == 4) return uniform ? sign_kernel<kLds, 1, 4> : sign_kernel<kLds, 0, 4>;
    if (share == 2) return uniform ? sign_kernel<kLds, 1, 2> : sign_kernel<kLds, 0, 2>;
    return uniform ? sign_kernel<kLds, 1, 1> : sign_kernel<kLds, 0, 1>;
}

static SignKernel sign_fn(int lds, int uniform, int share)
{
    return lds ? sign_fn_l<1>(uniform, share) : sign_fn_l<0>(uniform, share);
}

hipError_t launch_signs(const WalkArgs& a, const SignShape& sh, int uniform, int share, uint32_t grid, hipStream_t st)
{
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(sign_fn(sh.lds, uniform, share), dim3(grid), dim3(sh.threads), sh.bytes, st, a);
    return hipGetLastError();
}

int signs_occupancy(const SignShape& sh, int uniform, int share, int* wgs_per_cu)
{
    const void* fn = (const void*)sign_fn(sh.lds, uniform, share);
    int nb = 0;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSignLdsMost) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, (int)sh.threads, sh.bytes) != hipSuccess) {
        (void)hipGetLastError();
        return -1;
    }
    *wgs_per_cu = nb;
    return 0;
}

}  // namespace pw
