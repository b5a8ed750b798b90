// Host check of what the sign-table kernels read (pw_signtab.hpp). "degrees lo hi":
// prints "ok" when every degree of [lo, hi) is the whole number next to the
// reciprocal of its binary32 reciprocal, also with the reciprocal an ulp off on
// either side, else "bad d". "order n d_0 ... d_{n-1}", degrees descending: prints
// "ok words" when every node resolves through its packed block entry, and lies in
// the word and position that its run gives, else "bad x".
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "pw_signtab.hpp"

static unsigned degree_of(float inv, int ulps)
{
    float r = 1.0f / inv;
    if (ulps) r = std::nextafterf(r, ulps < 0 ? 0.0f : INFINITY);
    return (unsigned)(r + 0.5f);
}

int main()
{
    char what[16];
    while (std::scanf("%15s", what) == 1) {
        if (!std::strcmp(what, "degrees")) {
            unsigned lo, hi, d;
            if (std::scanf("%u %u", &lo, &hi) != 2) return 2;
            for (d = lo; d < hi; ++d) {
                const float inv = 1.0f / (float)d;
                if (degree_of(inv, -1) != d || degree_of(inv, 0) != d || degree_of(inv, 1) != d) break;
            }
            if (d < hi) std::printf("bad %u\n", d);
            else std::printf("ok\n");
            continue;
        }
        size_t n;
        if (std::scanf("%zu", &n) != 1) return 2;
        std::vector<uint32_t> rp(n + 1, 0u);
        for (size_t i = 0; i < n; ++i) {
            unsigned d;
            if (std::scanf("%u", &d) != 1) return 2;
            rp[i + 1] = rp[i] + d;
        }
        pw::SignOrder o;
        if (!pw::plan_sign_order(rp, &o)) {
            std::printf("nofit\n");
            continue;
        }
        std::vector<uint32_t> pos, blk, words;
        pw::build_sign_order(rp, o, &pos, &blk);
        const std::vector<uint32_t> entry = pw::pack_sign_blocks(blk);
        const std::vector<pw::SignRun> runs = pw::sign_runs(o, &words);
        size_t bad = entry.size() % 4 ? 0 : n, r = 0;
        for (size_t x = 0; x < n && bad == n; ++x) {
            while (runs[r + 1].first <= x) ++r;
            const uint32_t p = pos[x], b = p >> o.shift, w = runs[r].word + (p / 32 - runs[r].pos / 32);
            float inv;
            std::memcpy(&inv, &entry[2 * b + 1], 4);
            const unsigned d = degree_of(inv, 0);
            if (d != rp[x + 1] - rp[x] || entry[2 * b] + p * d != rp[x]) bad = x;
            if (p != runs[r].pos + (x - runs[r].first) || w >= words.size() || words[w] != p / 32) bad = x;
        }
        if (runs.back().word != words.size() || runs.back().first != n) bad = 0;
        if (bad < n) std::printf("bad %zu\n", bad);
        else std::printf("ok %zu\n", words.size());
    }
    return 0;
}
