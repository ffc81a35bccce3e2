// Prints what pf2_plan picks: one line "NT KS T split tiles pairs slices" for every "NT KS T split" on stdin (256 compute units).
#include <cstdio>

#include "prompt_plan.h"

int main()
{
    int NT, KS, T, split;
    while (std::scanf("%d %d %d %d", &NT, &KS, &T, &split) == 4) {
        const Pf2Plan p = pf2_plan(256, NT, KS, T, split != 0);
        std::printf("%d %d %d %d %d %d %d\n", NT, KS, T, split, pf2_variants[p.variant].ntw, pf2_variants[p.variant].pairs, p.slices);
    }
    return 0;
}
