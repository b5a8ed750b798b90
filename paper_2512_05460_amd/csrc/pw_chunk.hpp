// What the walk kernels of every table form share: the probes of a
// walk-sharing group, exact sums in LDS, the query's median, the claiming of
// chunks by persistent launches and the watchdog's flag.
#pragma once

#include "pw_device.hpp"
#include "pw_internal.hpp"

namespace pw {

// Probes [*kf, *kf + *sz) of walk-sharing group gi: groups of M probes inside
// each block of B (the last group of a block may be smaller).
__device__ __forceinline__ void group_probes(uint32_t gi, uint32_t B, uint32_t M, uint32_t gpb, uint32_t* kf,
                                             uint32_t* sz)
{
    const uint32_t blk = gi / gpb;
    const uint32_t j = gi - blk * gpb;
    *kf = blk * B + j * M;
    *sz = min(M, B - j * M);
}

__device__ __forceinline__ void lds_add_i128(unsigned long long* p, i128 v)
{
    const unsigned long long lo = (unsigned long long)(u128)v;
    const unsigned long long hi = (unsigned long long)((u128)v >> 64);
    const unsigned long long old = atomicAdd(p, lo);
    const unsigned long long carry = (old + lo < old) ? 1ull : 0ull;
    atomicAdd(p + 1, hi + carry);
}

// What the work groups of a query exchange while a launch runs are the words of
// its block sums, split-probe sums and counters, and each access to them is a
// read-modify-write at device scope, clearing included: there is one order of
// them per word, whatever XCD they come from, and each sees the value that the one
// before it left. Between words the order is the hardware's, not a fence's: a wave
// waits here until its atomics have been performed, so that they come before
// whatever another wave does once it has seen a counter that this one adds to
// next. Everything else a query leaves is read after the launch. (A device-scope
// fence would also write the XCD's whole L2 back and invalidate it: at L = 1 and
// R = 100 it made 480 us of what takes 261 us.)
__device__ __forceinline__ void atomics_performed()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// A 128-bit sum as its atomic additions have left it; its words are zero after
// that, for the next query of the slot or range. (Adding 0 instead would be a plain
// load: the compiler makes one of it.)
__device__ __forceinline__ i128 take_i128(unsigned long long* p)
{
    const unsigned long long lo = atomicExch(p, 0ull), hi = atomicExch(p + 1, 0ull);
    return (i128)(((u128)hi << 64) | (u128)lo);
}

// Median of the G block means (section 3.2, Algorithm 1 final loop), by the whole
// work group: a thread per block reads its sum and counts the smaller means.
// ys: kMaxG + 2 doubles of LDS. (By one thread the G reads, each a round trip to
// memory, followed one another.)
__device__ inline void finalize_query(const WalkArgs& A, const QueryDesc& d, double* ys)
{
    const uint32_t G = d.G, g = threadIdx.x;
    unsigned long long* bs = A.blocksum + (size_t)d.slot * A.gdim * 2;
    if (g < G) {
        const double y = (i128_to_f64(take_i128(bs + 2 * g)) * 0x1p-64) / (double)d.B;
        ys[g] = y;
        if (A.ybar_debug) A.ybar_debug[g] = y;
    }
    __syncthreads();
    if (g < G) {
        const double y = ys[g];
        uint32_t rank = 0;
        for (uint32_t i = 0; i < G; ++i) rank += ys[i] < y || (ys[i] == y && i < g) ? 1u : 0u;
        if (rank == (G - 1u) / 2u) ys[kMaxG] = y;
        if (rank == G / 2u) ys[kMaxG + 1] = y;
    }
    __syncthreads();
    if (g != 0) return;
    const double med = (G & 1u) ? ys[kMaxG] : 0.5 * (ys[kMaxG] + ys[kMaxG + 1]);
    A.beta[d.slot] = med;
    if (A.recycle) atomicExch(A.done + (size_t)d.slot * A.done_stride, 0u);
    if (A.comp_ring) {
        const uint32_t i = atomicAdd(A.comp_count, 1u);
        Completion c;
        c.slot = d.slot;
        c.pad = 0u;
        c.beta = med;
        A.comp_ring[i % A.comp_cap] = c;
    }
}

// The host watchdog's abort flag (host memory, read at system scope; the
// value is uniform over the work group once read by one thread, and a flag
// seen late only lets one more chunk run).
__device__ __forceinline__ bool abort_raised(const WalkArgs& A)
{
    return A.abort_flag != nullptr &&
           __hip_atomic_load(A.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0u;
}

// Part of a split group: add each probe's partial sums to its accumulator; the
// chunk that brings a probe's replica count to R forms its Q_R. acc holds the
// exact S1, S2 of the probes [k0, k0 + kc) over this chunk's pc replicas. flag:
// a word of LDS.
__device__ __forceinline__ void finish_parts(const WalkArgs& A, const QueryDesc& d, uint32_t k0, uint32_t kc,
                                             uint32_t pc, const unsigned long long* acc, double* ys, uint32_t* flag)
{
    if (threadIdx.x == 0) {
        uint32_t last = 0;
        for (uint32_t j = 0; j < kc; ++j) {
            const uint32_t k = k0 + j;
            const size_t pi = (size_t)d.psum_base + k;
            unsigned long long* ps = A.psum + pi * 4;
            atomic_add_i128(ps, (i128)(((u128)acc[4 * j + 1] << 64) | (u128)acc[4 * j]));
            atomic_add_i128(ps + 2, (i128)(((u128)acc[4 * j + 3] << 64) | (u128)acc[4 * j + 2]));
            atomics_performed();
            const uint32_t prev = atomicAdd(A.pcount + pi, pc);
            if (prev + pc == d.R) {
                // every part of this probe has been added
                const i128 S1 = take_i128(ps);
                const u128 S2 = (u128)take_i128(ps + 2);
                atomicExch(A.pcount + pi, 0u);
                const double Q = probe_q(S1, S2, d.R);
                if (A.q_debug) A.q_debug[k] = Q;
                atomic_add_i128(A.blocksum + ((size_t)d.slot * A.gdim + k / d.B) * 2, f64_to_i128_trunc(Q * 0x1p64));
                atomics_performed();
                const uint32_t old = atomicAdd(A.done + (size_t)d.slot * A.done_stride, 1u);
                if (old + 1u == d.K()) last = 1;
            }
        }
        *flag = last;
    }
    __syncthreads();
    const bool last = *flag != 0u;
    __syncthreads();
    if (last) finalize_query(A, d, ys);
    __syncthreads();
}

// Whole probes [k0, k0 + kc): each forms its Q_R from the exact sums in acc and
// adds it to its block; the one that completes the query forms the median.
__device__ __forceinline__ void finish_probes(const WalkArgs& A, const QueryDesc& d, uint32_t k0, uint32_t kc,
                                              const unsigned long long* acc, double* ys, uint32_t* flag,
                                              uint32_t threads)
{
    for (uint32_t j = threadIdx.x; j < kc; j += threads) {
        const i128 S1 = (i128)(((u128)acc[4 * j + 1] << 64) | (u128)acc[4 * j]);
        const u128 S2 = ((u128)acc[4 * j + 3] << 64) | (u128)acc[4 * j + 2];
        const double Q = probe_q(S1, S2, d.R);
        const uint32_t k = k0 + j;
        if (A.q_debug) A.q_debug[k] = Q;
        atomic_add_i128(A.blocksum + ((size_t)d.slot * A.gdim + k / d.B) * 2, f64_to_i128_trunc(Q * 0x1p64));
    }
    atomics_performed();
    __syncthreads();
    if (threadIdx.x == 0) *flag = atomicAdd(A.done + (size_t)d.slot * A.done_stride, kc) + kc == d.K() ? 1u : 0u;
    __syncthreads();
    const bool last = *flag != 0u;
    __syncthreads();
    if (last) finalize_query(A, d, ys);
    __syncthreads();
}

// Claim chunks from the queue of this XCD first, then from the others in turn.
// A queue seen empty stays empty (its cursor only grows), so each work group
// makes at most nqueues failed claims and every wave exits. Once its own queue
// is empty a work group reads the other cursors before it adds to them: at the
// end of a launch every work group would otherwise add to every cursor in
// vain, thousands of additions to a few words one after another.
// qstate: the current queue and the set of those found empty.
__device__ __forceinline__ void first_queue(const WalkArgs& A, uint32_t* qstate)
{
    uint32_t xcc = 0;
    if (A.nqueues > 1) asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    qstate[0] = (xcc & 15u) % A.nqueues;
    qstate[1] = 0;
}

__device__ __forceinline__ uint32_t claim_chunk(const WalkArgs& A, uint32_t* qstate)
{
    const uint32_t all = (1u << A.nqueues) - 1u;
    uint32_t ci = 0xFFFFFFFFu;
    uint32_t qi = qstate[0], empty = qstate[1];
    if (abort_raised(A)) empty = all;  // take no further chunk
    while (empty != all) {
        if (!(empty >> qi & 1u)) {
            const uint32_t beg = A.qoff[qi];
            const uint32_t c = atomicAdd(A.cursor + qi * A.cursor_stride, 1u);
            if (c < A.qoff[qi + 1] - beg) {
                ci = beg + c;
                break;
            }
            empty |= 1u << qi;
            for (uint32_t i = 0; i < A.nqueues; ++i)
                if (__hip_atomic_load(A.cursor + i * A.cursor_stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >=
                    A.qoff[i + 1] - A.qoff[i])
                    empty |= 1u << i;
        }
        qi = qi + 1 == A.nqueues ? 0u : qi + 1;
    }
    qstate[0] = qi;
    qstate[1] = empty;
    return ci;
}

}  // namespace pw
