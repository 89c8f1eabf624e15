// map_plan: prints what plan_map answers for "rows cols aligned16 transposed" lines on standard input, and what tiles_for_both
// makes of each line and the one before it
#include <cstdio>

#include "fxp_map_plan.h"

int main() {
    long long rows, cols;
    int aligned16, transposed;
    fxp::MapPlan before{};
    long long cols_before = 0;
    while (std::scanf("%lld %lld %d %d", &rows, &cols, &aligned16, &transposed) == 4) {
        const fxp::MapPlan p = fxp::plan_map(rows, cols, aligned16 != 0, transposed != 0);
        std::printf("%d %d %d %d %d %d %d\n", p.tc, p.passes, p.tiles, p.any, p.flat, p.tile_path,
                    cols_before != 0 && fxp::tiles_for_both(before, cols_before, p, cols));
        before = p;
        cols_before = cols;
    }
}
