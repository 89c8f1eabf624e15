// How a map launch cuts a tensor up: host arithmetic only, so that it can be checked without a device.
#pragma once
#include <cstdint>

namespace fxp {

struct MapPlan {
    int tc;          // tile columns
    int passes;      // 4, 2 or 1
    bool tiles;      // the tensor can be cut into tiles (their 32-bit addressing reaches all of it)
    bool any;        // rows that are not whole quads, or pointers off the 16-byte grid
    bool flat;       // one run of quads (no transposed copy)
    bool tile_path;  // the kernel of tiles and flat runs; false: the one-element-per-thread kernel
};

constexpr int64_t kFlatTileElements = 4096;                 // of one pass
constexpr int64_t kFlatMaxElements = int64_t{1} << 26;      // of a tensor of long rows

// aligned16: x and the copies that are wanted lie on the 16-byte grid; transposed: a transposed copy is wanted
inline MapPlan plan_map(int64_t rows, int64_t cols, bool aligned16, bool transposed) {
    MapPlan p;
    // tile width: 64 when that pads the rows less than 128 does (cols = 64, 192, ...)
    p.tc = ((cols + 63) / 64) * 64 < ((cols + 127) / 128) * 128 ? 64 : 128;
    p.any = cols % 4 != 0 || !aligned16;
    const int64_t tall = p.tc == 128 ? 128 : 256;   // rows of a 4-pass tile
    const int64_t tiles_c = (cols + p.tc - 1) / p.tc;
    auto tile_count = [&](int64_t passes) { return (rows + tall / 4 * passes - 1) / (tall / 4 * passes) * tiles_c; };
    p.tiles = rows > 0 && cols > 0 && cols < (int64_t{1} << 22) &&      // 32-bit offsets inside a tile
              rows < (int64_t{1} << 32) &&                              // and a 32-bit row count in the transposed copy's addressing
              (!p.any || cols >= 16) &&     // of a row shorter than a quarter of a tile most lanes would map nothing
              tile_count(1) < (int64_t{1} << 30);
    // Row-major only: flat, but tiles where a tensor of long rows is so large that it comes from HBM alone - their short
    // runs in many rows spread better (stochastic rounding, flat / tiles in us: 8192 x 2048 15.0 / 18.9, 8192 x 4096
    // 26.7 / 27.0, 12288 x 4096 39.7 / 39.4, 16384 x 4096 62.6 / 61.1, 16384 x 8192 129 / 120, 50000 x 2048 99.6 / 94.0; of
    // shorter rows 262144 x 256 62.3 / 63.5, 4194304 x 16 62.6 / 162).
    p.flat = !transposed && (!p.tiles || p.any || cols < 1024 || rows * cols < kFlatMaxElements);
    // four passes per tile when that still gives a thousand workgroups (four per CU), else two, else single-pass
    // tiles (a sweep of the threshold from 512 to 8192 moved whole-step times by under 3 %)
    auto count = [&](int64_t passes) {
        return p.flat ? (rows * cols + kFlatTileElements * passes - 1) / (kFlatTileElements * passes) : tile_count(passes);
    };
    p.passes = count(4) >= 1024 ? 4 : (count(2) >= 1024 ? 2 : 1);
    p.tile_path = p.flat ? rows > 0 && cols > 0 && count(1) < (int64_t{1} << 30) : p.tiles;
    return p;
}

// Two tensors of a launch, at least one of them planned flat: tiles for both where they are of one width, need no unaligned
// accesses and a flat one would fill seven eighths of its tiles - one body in the launch is less than two (layer steps, image
// flat / tiled in us: 32 x 28 x 28 x 128 -> 256 3x3 stride 2 57.5 / 56.2, 32 x 7 x 7 x 512 3x3 82.9 / 81.7), but a row of four
// channels leaves most of a tile empty (64 x 56 x 56 x 4 -> 128 1x1 stride 2 63.4 / 70.4, 2 x 512 x 512 x 4 -> 128 3x3 300 / 318).
inline bool tiles_for_both(const MapPlan& a, int64_t cols_a, const MapPlan& b, int64_t cols_b) {
    auto full = [](const MapPlan& p, int64_t cols) { return 8 * cols >= 7 * ((cols + p.tc - 1) / p.tc * p.tc); };
    return a.tiles && b.tiles && a.tc == b.tc && !a.any && !b.any && (!a.flat || full(a, cols_a)) && (!b.flat || full(b, cols_b));
}

}  // namespace fxp
