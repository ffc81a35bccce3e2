// Prints what pf2_plan picks: one line "NT KS T split tiles pairs slices" for every "NT KS T split" on stdin (256 compute units),
// or, with an argument, what tr_slices picks: "M N K tiles16 part_floats slices chunk" for every "M N K tiles16 part_floats".
#include <cstdio>

#include "prompt_plan.h"

int main(int argc, char **)
{
    if (argc > 1) {
        int M, N, K, tiles16;
        long part;
        while (std::scanf("%d %d %d %d %ld", &M, &N, &K, &tiles16, &part) == 5) {
            const TrSlices c = tr_slices(256, M, N, K, tiles16 != 0, (size_t)part);
            std::printf("%d %d %d %d %ld %d %d\n", M, N, K, tiles16, part, c.slices, c.chunk);
        }
        return 0;
    }
    int NT, KS, T, split;
    while (std::scanf("%d %d %d %d", &NT, &KS, &T, &split) == 4) {
        const Pf2Plan p = pf2_plan(256, NT, KS, T, split != 0);
        std::printf("%d %d %d %d %d %d %d\n", NT, KS, T, split, pf2_variants[p.variant].ntw, pf2_variants[p.variant].pairs, p.slices);
    }
    return 0;
}
