// Host check of the sign-table kernels' node order (pw_signtab.hpp): reads
// cases from stdin, one per line: "n d_0 ... d_{n-1}" with the degrees in
// descending order. For each it prints "ok shift positions" when every node's
// position is new, within range and resolves to the node's row offset and
// degree through its block's entry, else "bad x".
#include <cstdio>
#include <cstring>
#include <vector>

#include "pw_signtab.hpp"

int main()
{
    size_t n;
    while (std::scanf("%zu", &n) == 1) {
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
        std::vector<uint32_t> pos, blk;
        pw::build_sign_order(rp, o, &pos, &blk);
        std::vector<bool> seen(o.np, false);
        size_t bad = n;
        for (size_t x = 0; x < n && bad == n; ++x) {
            const uint32_t p = pos[x];
            if (p >= o.np || seen[p]) {
                bad = x;
                break;
            }
            seen[p] = true;
            const uint32_t* e = &blk[4 * (size_t)(p >> o.shift)];
            float inv;
            std::memcpy(&inv, e + 2, 4);
            if (p * e[1] + e[0] != rp[x] || e[1] != rp[x + 1] - rp[x] || inv != 1.0f / (float)e[1]) bad = x;
        }
        if (bad < n) std::printf("bad %zu\n", bad);
        else std::printf("ok %u %u\n", o.shift, o.np);
    }
    return 0;
}
