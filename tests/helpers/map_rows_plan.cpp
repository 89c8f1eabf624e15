// map_rows_plan: for "rows cols tr" lines on standard input the plan of a tensor's tiles of quads - tr 0: as the library chooses
// it, -1: of a small tensor - whether its scale is found by a scan, and the height of a
// launch with it as a flat run.  Checks id / quads over every id of a tile.
#include <cstdio>

#include "fxp_map_plan.h"

int main() {
    long long rows, cols;
    int tr;
    while (std::scanf("%lld %lld %d", &rows, &cols, &tr) == 3) {
        const fxp::RowsPlan p = tr < 0    ? fxp::plan_scan(rows, cols)
                                : tr == 0 ? fxp::plan_rows(rows, cols)
                                          : fxp::plan_rows(rows, cols, tr, fxp::rows_windows(cols));
        int exact = 1;
        for (uint32_t id = 0; id < p.tr * p.quads + 4096; ++id) exact &= static_cast<uint32_t>((uint64_t{id} * p.magic) >> 32) == id / p.quads;
        std::printf("%d %u %u %u %lld %d %d %d\n", p.tr, p.windows, p.width, p.quads, static_cast<long long>(p.blocks), exact,
                    fxp::scan_fits({rows, cols}, nullptr),
                    fxp::rows_height(fxp::plan_map(rows, cols, false, false), rows, cols));
    }
}
