// Host check of the vote for a launch's shape (pw_signtab.hpp): reads cases from
// stdin, one per line: "m shape_0 work_0 ... shape_{m-1} work_{m-1}", and prints
// the shape taken for each.
#include <cstdio>

#include "pw_signtab.hpp"

int main()
{
    size_t m;
    while (std::scanf("%zu", &m) == 1) {
        pw::ShapeVote v;
        for (size_t i = 0; i < m; ++i) {
            int shape;
            double work;
            if (std::scanf("%d %lf", &shape, &work) != 2) return 2;
            v.add(shape, work);
        }
        std::printf("%d\n", v.best());
    }
    return 0;
}
