// gemm_plan: for "reduce pieces splits 0" lines on standard input the lanes that share a piece in a sum of slices, for "tiles M N K" lines
// whether a product takes tiles of 64 x 64, without and with its largest magnitude, for "patches M Cout C" lines whether a 1x1 layer's weight gradient goes through stored patches, for "wgrad M Cout K" lines the cut of a convolution's weight gradient: pairs, tile rows, tiles, slices, pixels of a slice, bytes of the slices.
#include <cstdio>
#include <cstring>

#include "fxp_gemm_plan.h"

int main() {
    char what[16];
    long long a, b, c;
    while (std::scanf("%15s %lld %lld %lld", what, &a, &b, &c) == 4) {
        if (std::strcmp(what, "reduce") == 0) {
            std::printf("%d\n", fxp::reduce_lanes(a, b));
            continue;
        }
        if (std::strcmp(what, "patches") == 0) {
            std::printf("%d\n", fxp::one_tap_patches(a, b, c));
            continue;
        }
        if (std::strcmp(what, "tiles") == 0) {
            std::printf("%d %d\n", fxp::quarter_tiles(a, b, c, false), fxp::quarter_tiles(a, b, c, true));
            continue;
        }
        const fxp::WgradCut p = fxp::plan_conv_wgrad(a, b, c);
        std::printf("%d %d %d %d %lld %lld\n", p.pairs, p.bm, p.tiles_m * p.tiles_n, p.slices, static_cast<long long>(p.per_slice),
                    static_cast<long long>(p.ws_bytes));
    }
}
