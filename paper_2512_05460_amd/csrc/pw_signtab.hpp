// Node order, block table and launch shapes of the sign-table kernels (host
// side, no HIP; the kernels that read them are in pw_signs.hip).
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <vector>

namespace pw {

// A launch shape of the sign-table kernels for a graph and sharing class: one
// to four work groups per CU.
struct SignShape {
    int lds = 0;           // 1: the adjacency is staged in LDS
    uint32_t threads = 0;  // per work group; 0: the tables do not fit
    uint32_t per_cu = 0;   // work groups a CU holds at once
    uint32_t bytes = 0;    // dynamic LDS
    uint32_t T = 0;        // sign tables
};
constexpr int kSignShapes = 4;

// The one shape that a launch over several queries takes: the one that most of
// their scored steps, pairs x (L + 1), ask for, and never one that none of them
// asks for, which may be empty (threads = 0), not even where every count is 0.
struct ShapeVote {
    double steps[kSignShapes] = {};
    bool asked[kSignShapes] = {};
    void add(int shape, double work)
    {
        steps[shape] += work;
        asked[shape] = true;
    }
    int best() const
    {
        int b = 0;
        for (int i = 1; i < kSignShapes; ++i)
            if (asked[i] && (!asked[b] || steps[i] > steps[b])) b = i;
        return b;
    }
};

constexpr uint32_t kSignShiftMin = 4, kSignShiftMax = 9;

// Nodes are given in descending degree (row offsets rp[0..n]). Every run of
// equal degree starts a new block of 2^shift positions, so that a block has one
// degree; positions past a run's end are padding.
struct SignOrder {
    uint32_t shift = 0;
    uint32_t np = 0;             // positions, a multiple of 16
    uint32_t nblk = 0;           // blocks
    std::vector<uint32_t> run;   // first storage id of each run, then n
};

// The block size for which the block table (8 bytes a block) and four sign
// tables (a bit a position each) take least; false beyond 2^24 positions,
// which the 24-bit products of the kernels could not hold.
inline bool plan_sign_order(const std::vector<uint32_t>& rp, SignOrder* o)
{
    const size_t n = rp.size() - 1;
    o->run.clear();
    for (size_t i = 0; i < n; ++i)
        if (i == 0 || rp[i + 1] - rp[i] != rp[i] - rp[i - 1]) o->run.push_back((uint32_t)i);
    o->run.push_back((uint32_t)n);
    uint64_t best = ~uint64_t(0);
    for (uint32_t s = kSignShiftMin; s <= kSignShiftMax; ++s) {
        uint64_t blocks = 0;
        for (size_t r = 0; r + 1 < o->run.size(); ++r)
            blocks += ((uint64_t)(o->run[r + 1] - o->run[r]) + (1u << s) - 1) >> s;
        const uint64_t np = blocks << s, bytes = 8 * blocks + np / 2;
        if (np <= (1u << 24) && bytes < best) {
            best = bytes;
            o->shift = s;
            o->np = (uint32_t)np;
            o->nblk = (uint32_t)blocks;
        }
    }
    return best != ~uint64_t(0);
}

// Where each run lies: its first storage id, first position, and first word of 32
// positions among those that hold nodes; then {n, ~0, the number of words}.
struct SignRun {
    uint32_t first, pos, word;
};

inline std::vector<SignRun> sign_runs(const SignOrder& o, std::vector<uint32_t>* words)
{
    std::vector<SignRun> runs;
    words->clear();
    uint32_t x0 = 0;
    for (size_t r = 0; r + 1 < o.run.size(); ++r) {
        const uint32_t len = o.run[r + 1] - o.run[r];
        uint32_t w = x0 / 32;
        if (!words->empty() && words->back() == w) ++w;  // begins in the last one's second half
        runs.push_back(SignRun{o.run[r], x0, (uint32_t)words->size() - (w - x0 / 32)});
        for (; w <= (x0 + len - 1) / 32; ++w) words->push_back(w);
        x0 += ((len + (1u << o.shift) - 1) >> o.shift) << o.shift;
    }
    runs.push_back(SignRun{o.run.back(), ~0u, (uint32_t)words->size()});
    return runs;
}

// pos[storage id] (unless null) and the block entries {base, d, bits of 1.0f/d, 0}:
// position x of a block has row offset base + x d (32-bit arithmetic, base may wrap).
inline void build_sign_order(const std::vector<uint32_t>& rp, const SignOrder& o, std::vector<uint32_t>* pos,
                             std::vector<uint32_t>* blk)
{
    if (pos) pos->resize(rp.size() - 1);
    blk->assign((size_t)o.nblk * 4, 0u);
    uint32_t at = 0;  // next block
    for (size_t r = 0; r + 1 < o.run.size(); ++r) {
        const uint32_t f = o.run[r], e = o.run[r + 1], d = rp[f + 1] - rp[f], x0 = at << o.shift;
        if (pos)
            for (uint32_t i = f; i < e; ++i) (*pos)[i] = x0 + (i - f);
        const float inv = 1.0f / (float)d;
        const uint32_t nb = (e - f + (1u << o.shift) - 1) >> o.shift, base = rp[f] - x0 * d;
        for (uint32_t b = 0; b < nb; ++b) {
            uint32_t* w = blk->data() + 4 * (size_t)(at + b);
            w[0] = base;
            w[1] = d;
            memcpy(w + 2, &inv, 4);
        }
        at += nb;
    }
}

// The entries as the kernels read them, {base, bits of 1.0f/d}, an even number.
// They take d as the whole number next to the reciprocal of 1.0f/d, which holds
// below 2^20.
inline std::vector<uint32_t> pack_sign_blocks(const std::vector<uint32_t>& blk)
{
    std::vector<uint32_t> entry((blk.size() / 4 + 1) / 2 * 4, 0u);
    for (size_t b = 0; b < blk.size() / 4; ++b) {
        entry[2 * b] = blk[4 * b];
        entry[2 * b + 1] = blk[4 * b + 2];
    }
    return entry;
}

}  // namespace pw
