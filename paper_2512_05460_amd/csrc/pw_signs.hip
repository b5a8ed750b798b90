// Walk kernels that score against sign tables in LDS.
//
// A probe's sign z^(k)(x) is a fixed function of the node. A chunk scores each
// of its probes 2 R (L + 1) times, and where that is more often than the graph
// has nodes it is cheaper to evaluate the Feistel permutation and the hash once
// per node into a table in LDS and let the walks look the sign up: 23
// instructions per walk step instead of 118. The tables are indexed by the
// node's position in the kernels' own tables, so the walks need neither the
// caller's id nor a row table from memory whatever layout the graph was loaded
// in. Two forms:
//
//   * Small graphs (kLds): row offset and degree of every node (4 bytes) and the
//     whole adjacency (2 bytes an entry) are staged in LDS, and a table holds
//     z / d as binary32. A step is three LDS reads and 14 instructions.
//   * Larger ones: nodes are stored in descending degree, each run of equal
//     degree padded to whole blocks of 2^shift positions, so a block has one
//     degree d and a node x of it has row offset base + x d. One LDS read of
//     the block's entry {base, d, bits of 1.0f/d} resolves a node: no search,
//     no division, no second dependent read from memory. A step reads one
//     neighbour position, 3 bytes, from memory (an L2 hit up to about 1.3
//     million adjacency entries); a table holds two bits a node.
//
// The walks, their random streams, the order of the binary32 sums and all
// results are those of the other kernels.
#include "pw_chunk.hpp"
#include "pw_device.hpp"
#include "pw_internal.hpp"

namespace pw {

// Dynamic LDS of a work group, in this order.
struct SignLds {
    uint4* blk;                 // nblk block entries; kLds: rows, then the adjacency
    unsigned long long* acc;    // T x {S1, S2}
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
        const uint4 e = M.blk[x >> S.shift];
        return SignNode<0>{x, umul24(x, e.y) + e.x, e.y, __uint_as_float(e.z)};
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

// acc + z(x) / d. From the two-bit table z in {-1, 0, 1} is exact, so the fused
// form rounds as the plain sum does; z = 0 leaves acc as it is (acc is never
// -0). The first of a word's 16 positions is in its top bits.
template <int kLds>
__device__ __forceinline__ float sign_add(const uint32_t* tab, const SignNode<kLds>& w, float acc)
{
    if constexpr (kLds) {
        return __fadd_rn(acc, *reinterpret_cast<const float*>(reinterpret_cast<const char*>(tab) + w.x4));
    } else {
        const int z = (int)(tab[w.x >> 4] << ((2u * w.x) & 31u)) >> 30;
        return __builtin_fmaf((float)z, w.inv, acc);
    }
}

// Fills the tables of probes [kA, kA + kn): each wave takes 64 words of one
// probe at a time (its keys are wave-uniform).
template <int kLds>
__device__ __forceinline__ void sign_build(const SignTables& S, const SignLds& M, const Domain& dom, const QueryDesc& d,
                                           uint32_t kA, uint32_t kn)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
    const uint32_t words = kLds ? S.tabw : S.words;
    const uint32_t segs = (words + 63u) >> 6;
    uint32_t cur = 0xFFFFFFFFu;
    Probe pr{};
    for (uint32_t u = wave; u < kn * segs; u += nw) {
        const uint32_t j = u / segs;
        if (j != cur) {
            pr = make_probe(d.seed_lo, d.seed_hi, d.uid, kA + j, dom.n);
            cur = j;
        }
        const uint32_t w = (u - j * segs) * 64u + lane;
        if (w >= words) continue;
        if constexpr (kLds) {
            uint32_t y;
            const uint32_t deg = reinterpret_cast<const uint32_t*>(M.blk)[w] >> 16;
            M.tab[j * S.tabw + w] =
                __float_as_uint(__fmul_rn((float)probe_value(w, pr, dom, &y), __fdiv_rn(1.0f, (float)deg)));
        } else {
            // a quarter of 64 words' ids at a time, one after another
            const uint4* ids = reinterpret_cast<const uint4*>(S.pid) + (size_t)(u - j * segs) * 256u + lane;
            uint32_t word = 0;
#pragma unroll 1
            for (uint32_t i = 0; i < 4; ++i) {
                const uint4 v = ids[64u * i];
                // four permutations at once; the few values that land past n are walked on
                uint32_t y[4] = {feistel_once(v.x, pr, dom), feistel_once(v.y, pr, dom), feistel_once(v.z, pr, dom),
                                 feistel_once(v.w, pr, dom)};
                while (max(max(y[0], y[1]), max(y[2], y[3])) >= dom.n) {
#pragma unroll
                    for (int h = 0; h < 4; ++h)
                        if (y[h] >= dom.n) y[h] = feistel_once(y[h], pr, dom);
                }
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const uint32_t neg = hash_bit(pr, y[h] >> 1) ^ (y[h] & 1u);
                    word = (word << 2) | (y[h] >= pr.zlo ? 0u : 2u * neg + 1u);  // 1, -1 as 3, or 0
                }
            }
            M.tab[j * S.tabw + S.pid[1024u * segs + w]] = word;
        }
    }
}

// U_p of replica p for the m probes of a group, whose tables start at tab (the
// streams are keyed by kw, the group's first probe). The two neighbour reads of
// a step are issued before the nodes just left are scored.
template <int kLds, int kShare>
__device__ __forceinline__ void sign_pair(const SignTables& S, const SignLds& M, const uint32_t* tab, uint32_t m,
                                          SignNode<kLds> s, SignNode<kLds> t, int L, uint32_t p, uint32_t kw, uint32_t uid,
                                          uint32_t slo, uint32_t shi, float* U)
{
    float a[kShare], b[kShare];
#pragma unroll
    for (int j = 0; j < kShare; ++j) a[j] = b[j] = 0.0f;
    auto score = [&]() {
#pragma unroll
        for (int j = 0; j < kShare; ++j) {
            if (kShare == 1 || (uint32_t)j < m) {
                a[j] = sign_add<kLds>(tab + j * S.tabw, s, a[j]);
                b[j] = sign_add<kLds>(tab + j * S.tabw, t, b[j]);
            }
        }
    };
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
    const uint32_t per_phase = max(1u, S.T / M_);
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
        sign_build<kLds>(S, M, dom, d, kA, kn);
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
                if (p < pend) {
                    float U[kShare];
                    sign_pair<kLds, kShare>(S, M, M.tab + (kf - kA) * S.tabw, m, s0, t0, d.L, p, kf, d.uid, d.seed_lo,
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
                float U[kShare];
                sign_pair<kLds, kShare>(S, M, M.tab + (kf - kA) * S.tabw, m, s0, t0, d.L, p, kf, d.uid, d.seed_lo,
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
    const uint32_t staged = kLds ? (S.nblk + S.idw) / 4u : S.nblk;
    M.blk = reinterpret_cast<uint4*>(lds);
    M.acc = reinterpret_cast<unsigned long long*>(M.blk + staged);
    M.tab = reinterpret_cast<uint32_t*>(M.acc + 4u * S.T);
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
