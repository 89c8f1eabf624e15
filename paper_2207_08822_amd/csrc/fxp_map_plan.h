// How a map launch cuts a tensor up: host arithmetic only, so that it can be checked without a device.
#pragma once
#include <cstdint>
#include <initializer_list>

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

// ---- tiles of quads (fxp_map_rows.hip) ----
constexpr uint32_t kRowsWidth = 128;                  // most columns of a window
// A tensor whose scale every workgroup works out for itself, 64 bytes a clock from L2: small tiles, many of them, but no more
// workgroups than CUs if it can be, since each CU reads the tensor once per workgroup.  Beyond some 100000 elements that takes longer
// than a reduction launch (steps of n^3 launched one by one, two launches / scan in us: 256 30 / 21.0, 300 26.8 / 22.2, 330 28.0 / 25.5,
// 362 29.8 / 31.0, 400 26.4 / 30.8; replayed from a graph: 300 22.0 / 20.7, 320 20.6 / 21.0, 336 20.6 / 21.4).  A single
// tensor wanted row-major only loses from 80 K elements on in a graph (133 x 858 6.2 / 6.9) what it gains launched by itself (115 x
// 968 14.3 / 11.4).
constexpr int64_t kScanMaxElements = 112 * 1024;

struct RowsPlan {
    int tr;                          // rows of a tile
    uint32_t windows, width;         // of a row: windows of `width` columns, the last one perhaps of fewer
    uint32_t quads, magic;           // most quads that a window meets in a row; id / quads = (id * magic) >> 32 for ids of a tile
    int64_t blocks;
};

// `windows` of a size (of any tensor of fewer than 2^22 columns), none wider than the stage of the kernel that they are for
inline RowsPlan plan_rows(int64_t rows, int64_t cols, int tr, int64_t windows) {
    RowsPlan p;
    p.tr = tr;
    int64_t width = (cols + windows - 1) / windows;
    if (cols % 4 == 0) width = (width + 3) / 4 * 4;               // whose quads then begin with them
    p.windows = static_cast<uint32_t>((cols + width - 1) / width);
    p.width = static_cast<uint32_t>(width);
    p.quads = cols % 4 == 0 ? p.width / 4 : (p.width + 6) / 4;
    if (p.quads < 2) p.quads = 2;                                 // (of one, the reciprocal has 33 bits)
    p.magic = 0xffffffffu / p.quads + 1;
    p.blocks = (rows + tr - 1) / tr * p.windows;
    return p;
}

// Windows of a row: 128 columns, or 125 where rows are not whole quads - the most that meet no more than 32 quads, so that 32 rows are
// one round of four quads a thread (with 33 every height took a round more for next to nothing, both copies: 12608 x 1001 21.8 -> 19.4
// us, 6000 x 1001 12.1 -> 11.1, 64 x 50257 10.6 -> 7.5, 1379 x 1001 6.6 -> 5.1).
inline int64_t rows_windows(int64_t cols) {
    const int64_t most = cols % 4 == 0 ? kRowsWidth : kRowsWidth - 3;
    return (cols + most - 1) / most;
}

// Tall tiles write long runs of the transposed copy, but a few hundred of them leave CUs with one tile more than others, and rounds of
// 1024 quads that the rows of a window do not fill leave lanes without one: the height and the windows - up to two more than need be -
// whose tiles fill 256 CUs and their rounds best, a halving counted as an eighth lost (both copies, heights and windows by the CUs alone
// / so, in us: 12608 x 1001 19.2 / 17.9, 25000 x 301 13.1 / 12.0, 28800 x 150 10.1 / 8.8, 70001 x 17 7.0 / 5.6, 6000 x 1001 11.0 / 12.1;
// rounding to nearest 28800 x 150 7.3 / 6.7, 9456 x 257 5.2 / 4.7); 32 rows and no window more below two tiles a CU.
inline RowsPlan plan_rows(int64_t rows, int64_t cols) {
    const int64_t windows = rows_windows(cols);
    RowsPlan best = plan_rows(rows, cols, 32, windows);
    const int64_t most = windows + (best.blocks < 512 ? 0 : 2);
    double best_score = 0.0, weight = 1.0;
    for (int tr : {128, 64, 32}) {
        for (int64_t w = windows; w <= most && (w == windows || cols >= 16 * w); ++w) {
            const RowsPlan p = plan_rows(rows, cols, tr, w);
            const int64_t lanes = (static_cast<int64_t>(tr) * p.quads + 1023) / 1024 * 1024 * ((p.blocks + 255) / 256 * 256);
            const double score = weight * static_cast<double>(rows * cols / 4) / static_cast<double>(lanes);
            if (p.blocks >= 512 && score > best_score) {
                best = p;
                best_score = score;
            }
        }
        weight *= 0.87;
    }
    return best;
}

// ... and what a flat run beside them has in place of rows, 32 a pass, is for as many workgroups as its own plan wants (the image
// of 4 x 224 x 224 x 3 beside the weights of its layer, as 37 workgroups of 16384 elements 9.5 us, as 147 5.0).
inline int rows_height(const MapPlan& p, int64_t rows, int64_t cols) { return p.flat ? 32 * p.passes : plan_rows(rows, cols).tr; }

// Tiles of about 1024 elements, so that a tensor of the limit is 112 of them: 32 rows, and columns to match where there are fewer
// (scale + map in us, two launches / scan with 32 columns / so: 8 x 12288 6.6 / 9.3 / 6.2, 4 x 16384 6.4 / 7.5 / 5.1, 1 x 32768
// 6.3 / 8.8 / 4.3).
inline int scan_width_log2(int64_t rows) { return rows > 16 ? 5 : rows > 8 ? 6 : 7; }
inline RowsPlan plan_scan(int64_t rows, int64_t cols) {
    const int shift = scan_width_log2(rows);
    return plan_rows(rows, cols, 32, (cols + (1 << shift) - 1) >> shift);
}

// Whether `blocks` workgroups together, each for the scale of a tensor of at most `elements`, read little enough: what a CU reads is
// what bounds them (scan of 1 x 114688 by 3584 workgroups 55.8 us, two launches 8.4; 2 x 50257, 1571 workgroups, 29.5 / 9.6; 8 x 12288,
// 384 workgroups, 9.3 / 6.6).
inline bool scan_pays(int64_t elements, int64_t blocks) { return (blocks + 255) / 256 * elements <= kScanMaxElements; }
inline bool scan_takes(int64_t rows, int64_t cols) {
    return rows > 0 && cols >= 16 && rows <= kScanMaxElements && cols <= kScanMaxElements && rows * cols <= kScanMaxElements;
}

// One tensor or two in a launch.  (Asked before every call's maps: no division where the widest windows already are one round.)
struct ScanSize {
    int64_t rows, cols;
};
inline bool scan_fits(ScanSize a, const ScanSize* b) {
    if (!scan_takes(a.rows, a.cols) || (b && !scan_takes(b->rows, b->cols))) return false;
    auto at_most = [](const ScanSize& t) {
        const int shift = scan_width_log2(t.rows);
        return ((t.rows + 31) >> 5) * ((t.cols + (1 << shift) - 1) >> shift);
    };
    if (at_most(a) + (b ? at_most(*b) : 0) <= 256) return true;
    const int64_t na = a.rows * a.cols, nb = b ? b->rows * b->cols : 0;
    return scan_pays(na > nb ? na : nb, plan_scan(a.rows, a.cols).blocks + (b ? plan_scan(b->rows, b->cols).blocks : 0));
}

}  // namespace fxp
