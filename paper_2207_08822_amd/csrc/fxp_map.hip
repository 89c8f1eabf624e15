// Linear fixed-point mapping fp32 -> int8 (paper Sec. 3.1) with the stochastic
// rounding of App. A.1 (Fig. 4): the 24-bit mantissa, shifted right by
// e_max - e, is cut after bits-1 magnitude bits and rounded up iff a random
// number is below the bits cut off.
//
// Kernel shape (HBM-bound by intent: 4 B read, 1 B written per copy per element;
// the Philox rounds make VALU the close second):
//   * one block = one 128 x 128 tile; each thread owns 4 x 4 element blocks, read
//     as four 16-byte loads along rows (one Philox call per load);
//   * q is written as packed dwords straight from registers (128 B per row per
//     half-wave);
//   * for the transposed copy the 4 x 4 block is transposed in registers, staged in
//     LDS as [col][row] bytes and written out in 16-byte pieces along rows of qT,
//     so both copies carry the same rounding decisions and both stores coalesce;
//   * the final step of the scale reduction (max over <= 1024 block maxima) can be
//     folded in, which saves a launch per tensor.
// Rows that are not whole quads, and bases off the 16-byte grid, take tiles of quads (fxp_map_rows.hip), as do small tensors,
// whose scale is found in the same launch; a tensor that is wanted row-major only is one flat run of quads (map_flat_body) up to
// a size; the one-element-per-thread kernel is left for what none of them reaches.
// The random word of element i is word (i mod 4) of Philox-4x32-10 with key = seed
// and counter = (i / 4, stream_id): nothing depends on the launch geometry.
#include <algorithm>

#include "fxp_internal.h"
#include "fxp_map_device.h"
#include "fxp_map_plan.h"

namespace fxp {

template <int V>
using IC = std::integral_constant<int, V>;

// One tensor of a map launch.  A launch carries up to two (the activation and the weight of a forward pass):
// the first `blocks` workgroups belong to job 0, the rest to job 1.
struct MapJob {
    const uint32_t* x;
    int64_t rows, cols;
    const int32_t* e_in;
    const uint32_t* partials;
    int n_partials;
    int32_t* e_out;
    int8_t* q;
    int8_t* qT;
    uint32_t sid0, sid1;
    int tiles_c;
    int flat;               // row-major copy only: rows and columns do not matter (map_flat_body)
    unsigned blocks;
    unsigned xcd_blocks;    // leading workgroups whose tiles are numbered per XCD (see tile_of_workgroup)
    // scale taken as a guess (see k_map_tile_guess): where the guess comes from, where the largest exponents that the
    // workgroups of the guessing launch met go, how many, and the word that records which guess the tensor was mapped with
    // (0 = none)
    const int32_t* e_guess;
    uint8_t* guess_maxima;
    int guess_blocks;
    int32_t* guess_used;
};
struct MapJobs {
    MapJob j[2];
};

// Row block and column block of workgroup `bid` of a tensor.  Plain numbering walks the column tiles of a row
// block first.  Where a row is not a whole number of 128-byte lines, neighbouring column tiles share the lines
// their boundary falls into, and workgroups are dealt to the eight XCDs in turn, each with an L2 of its own: such a
// tensor numbers its tiles so that the column tiles of one row block are eight workgroups apart - the same XCD,
// one after the other - and the shared lines come from that L2 the second time (row blocks beyond the last
// whole group of eight keep the plain numbering).
__device__ inline void tile_of_workgroup(const MapJob& J, unsigned bid, unsigned* rb, unsigned* cb) {
    const unsigned tc = static_cast<unsigned>(J.tiles_c);
    if (bid < J.xcd_blocks) {
        const unsigned group = bid / (8u * tc), local = bid % (8u * tc);
        *rb = group * 8u + (local & 7u);
        *cb = local >> 3;
    } else {
        const unsigned i = bid - J.xcd_blocks;
        *rb = J.xcd_blocks / tc + i / tc;
        *cb = i % tc;
    }
}

// One tile of TC columns (128, or 64 for tensors whose width pads less that way: head width 64 of the
// attention operands) and TR = 1024 / TC * 4 * PASSES rows: every thread owns 4 x 4 elements per pass, the 256
// threads of a pass cover 32 x 128 or 64 x 64.  PASSES = 4 for large tensors, 2 or 1 when the tensor is too small
// to fill the chip with the taller tiles.  EDGE = the tile sticks out of the tensor: loads are clamped to valid
// addresses and stores are predicated; interior tiles carry no bounds code at all.  All
// per-thread addressing is a 32-bit element offset from the tile's (wave-uniform) origin.
// GUESS: the scale is not resolved from block maxima but given (e_given; do_map = false: there is none, only the
// maximum is wanted), and the largest magnitude bits of the tile are accumulated into tile_max (clamped loads
// of an edge tile repeat elements of the tensor, which a maximum does not mind).
template <bool STOCH, bool EDGE, int PASSES, int TC, bool GUESS = false>
__device__ inline void map_tile_body(const uint32_t* __restrict__ x, int64_t rows, int64_t cols, const MapJob& J, int bits,
                                     bool publish, uint32_t* red, int8_t* __restrict__ q, int8_t* __restrict__ qT,
                                     uint32_t key0, uint32_t key1, uint32_t sid0, uint32_t sid1, int64_t r0, int64_t c0,
                                     uint32_t* stage, int e_given = 0, bool do_map = true, uint32_t* tile_max = nullptr) {
    constexpr int CG = TC / 4;                    // groups of 4 columns
    constexpr int RGP = kMapThreads / CG;         // groups of 4 rows per pass
    constexpr int TR = 4 * RGP * PASSES;          // rows of the tile
    constexpr int TS = RGP * PASSES + 1;          // dwords per staged column (TR row bytes + 4 pad)
    int tid = threadIdx.x;
    // (in the loop over tiles: nothing that follows from the thread is kept from one tile to the next, which took 173 registers)
    if (GUESS) asm volatile("" : "+v"(tid));
    const int cg = tid % CG;                      // group of 4 columns
    const int rgl = tid / CG;                     // group of 4 rows within a pass
    const uint32_t ucols = static_cast<uint32_t>(cols);
    const int64_t origin = r0 * cols + c0;        // element index of the tile's first element (multiple of 4)
    const uint32_t* xt = x + origin;
    int8_t* qt = q ? q + origin : nullptr;
    const uint64_t blk0 = static_cast<uint64_t>(origin) >> 2;
    const int rows_here = EDGE ? static_cast<int>(min<int64_t>(TR, rows - r0)) : TR;
    const int cols_here = EDGE ? static_cast<int>(min<int64_t>(TC, cols - c0)) : TC;
    const bool col_ok = !EDGE || 4 * cg < cols_here;
    const uint32_t col_ld = EDGE ? static_cast<uint32_t>(min(4 * cg, cols_here - 4)) : 4 * cg;

    // PASSES passes of 4 * RGP rows.  The loads of pass p+1 are issued before the arithmetic of pass
    // p, so a block keeps the memory pipe busy while it runs its Philox rounds.
    auto load_pass = [&](int p, uint4 (&v)[4]) {
        const int lrow = 4 * (p * RGP + rgl);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int rr = EDGE ? min(lrow + k, rows_here - 1) : lrow + k;
            v[k] = *reinterpret_cast<const uint4*>(xt + static_cast<uint32_t>(rr) * ucols + col_ld);
        }
    };
    uint4 cur[4], nxt[4];
    const bool given = GUESS || e_given != 0;
    const uint32_t share = given ? 0u : partials_share(J.partials, J.n_partials);
    load_pass(0, cur);
    // the scale is resolved (block maxima re-read and reduced) while the first loads are in flight
    const MapCfg cfg = make_cfg(given ? e_given : resolve_scale(J.e_in, J.partials, share, J.e_out, red, publish), bits);
    const bool scale_ok = cfg.e_max >= 25 && cfg.e_max < 255;
    const uint32_t over_bits = ~cfg.sat;          // a fast-path result with any of these set needs saturation
    uint32_t seen = 0;                             // GUESS: largest magnitude bits this thread has loaded
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int rg = p * RGP + rgl;              // group of 4 rows
        const int lrow = 4 * rg;
        if (p + 1 < PASSES) load_pass(p + 1, nxt);
        if (GUESS) {
#pragma unroll
            for (int k = 0; k < 4; ++k) seen = max(seen, absmax4(cur[k]));
            if (!do_map) {                         // workgroup-uniform: no scale to map with, the maximum is all
#pragma unroll
                for (int k = 0; k < 4; ++k) cur[k] = nxt[k];
                continue;
            }
        }
        auto words_of = [&](int k) {
            if (!STOCH) return make_uint4(0, 0, 0, 0);
            const uint64_t blk = blk0 + ((static_cast<uint32_t>(lrow + k) * ucols + 4 * cg) >> 2);
            return philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(blk >> 32), sid0, sid1, key0, key1);
        };
        uint32_t o[4];
        uint32_t q_or = 0;
        uint64_t bad = 0;                          // wave-uniform: any lane with an uncovered element
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = map_quad_fast<STOCH>(cur[k], words_of(k), cfg, q_or, bad);
        if (!scale_ok || bad != 0 || (q_or & over_bits)) {
            // rare: an element above the scale, a saturating result, a non-finite input or a tiny
            // scale somewhere in this 4 x 4 block: redo it with the complete per-element path
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = map_quad_full<STOCH>(cur[k], words_of(k), cfg);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (qt != nullptr && col_ok && (!EDGE || lrow + k < rows_here))
                *reinterpret_cast<uint32_t*>(qt + static_cast<uint32_t>(lrow + k) * ucols + 4 * cg) = o[k];
        if (qT != nullptr) {
            uint32_t t[4];                          // t[c] = column c of the block, rows in ascending byte order
            transpose4x4(o, t);
#pragma unroll
            for (int c = 0; c < 4; ++c) stage[(4 * cg + c) * TS + rg] = t[c];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) cur[k] = nxt[k];
    }
    if (GUESS) *tile_max = max(*tile_max, seen);
    if (qT == nullptr || (GUESS && !do_map)) return;
    __syncthreads();
    int8_t* qTt = qT + c0 * rows + r0;             // element [c0][r0] of the transposed copy
    const uint32_t urows = static_cast<uint32_t>(rows);
    constexpr int PIECES = TR / 16;                // 16 rows of one column = 16 contiguous bytes of qT
    constexpr int ROUNDS = (TC * PIECES + kMapThreads - 1) / kMapThreads;
    // Rows that are whole pieces have a loop of their own, and that of edge tiles is not unrolled: every map kernel holds them all
    // (with one unrolled loop for either, k_map_tile_guess lost 2 % of a step: 12608 x 768 x 2304 164.0 -> 167.1 us).
    if ((rows & 15) == 0) {
#pragma unroll
        for (int it = 0; it < ROUNDS; ++it) {
            const int id = it * kMapThreads + tid;
            const int c = id / PIECES, ch = id % PIECES;
            if (c < TC && (!EDGE || (c < cols_here && 16 * ch < rows_here))) {
                const uint32_t* src = stage + c * TS + 4 * ch;
                *reinterpret_cast<uint4*>(qTt + static_cast<uint64_t>(c) * urows + 16 * ch) =
                    make_uint4(src[0], src[1], src[2], src[3]);
            }
        }
        return;
    }
    // ... any others take 16 bytes at any alignment, and their last bytes one by one
    constexpr int UNROLLED = EDGE ? 1 : ROUNDS;
#pragma unroll UNROLLED
    for (int it = 0; it < ROUNDS; ++it) {
        const int id = it * kMapThreads + tid;
        const int c = id / PIECES, ch = id % PIECES;
        if (c < TC && (!EDGE || (c < cols_here && 16 * ch < rows_here))) {
            const uint32_t* src = stage + c * TS + 4 * ch;
            int8_t* dst = qTt + static_cast<uint64_t>(c) * urows + 16 * ch;
            if (!EDGE || 16 * ch + 16 <= rows_here) {
                *reinterpret_cast<Bytes16*>(dst) = Bytes16{src[0], src[1], src[2], src[3]};
            } else {
                for (int r = 0; 16 * ch + r < rows_here; ++r) dst[r] = static_cast<int8_t>(src[r >> 2] >> (8 * (r & 3)));
            }
        }
    }
}

// the scale that the guessing launch has seen: largest of at most kGuessBlocks exponents, sixteen a thread
__device__ inline int scale_of_guess(const MapJob& J, uint32_t* red) {
    uint32_t m = 0;
    const int first = 16 * threadIdx.x;
    if (first < J.guess_blocks) {
        const uint4 v = reinterpret_cast<const uint4*>(J.guess_maxima)[threadIdx.x];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (first + k < J.guess_blocks) m = max(m, (w[k >> 2] >> (8 * (k & 3))) & 0xffu);
    }
    return max(1, static_cast<int>(block_max(m, red)));
}

// FLAT: a launch with a flat tensor in it.  (A parameter: with the flat body in every instantiation the tiles of an aligned
// tensor ran at lower occupancy or spilled, 159744 x 208 both copies 39.1 -> 40.0 us.)
template <bool STOCH, int PASSES, int TC, bool FLAT>
__global__ __launch_bounds__(kMapThreads) void k_map_tile(const MapJobs jobs, uint32_t key0, uint32_t key1, int bits) {
    constexpr int RGP = kMapThreads / (TC / 4);
    constexpr int TR = 4 * RGP * PASSES;
    __shared__ uint32_t stage[TC * (RGP * PASSES + 1)];
    __shared__ uint32_t red[kMapThreads / 64];
    const bool second = blockIdx.x >= jobs.j[0].blocks;            // workgroup-uniform
    const MapJob& J = jobs.j[second ? 1 : 0];
    const unsigned bid = blockIdx.x - (second ? jobs.j[0].blocks : 0u);
    int e_true = 0;
    if (J.guess_used != nullptr) {
        // this launch follows k_map_tile_guess: the tensor is already mapped if the guess was its scale - then
        // the scale is published and nothing else is left to do; otherwise the tile is mapped now
        e_true = scale_of_guess(J, red);
        if (bid == 0 && threadIdx.x == 0) J.e_out[0] = e_true;
        if (J.guess_used[0] == e_true) return;
    }
    if (FLAT && J.flat) {
        const uint64_t first = static_cast<uint64_t>(bid) * (4 * kMapThreads * PASSES);
        const uint64_t whole = static_cast<uint64_t>(J.rows) * static_cast<uint64_t>(J.cols) >> 2;
        if (first + 4 * kMapThreads * PASSES <= whole) map_flat_body<STOCH, PASSES, false>(J, bits, bid == 0, red, key0, key1, first);
        else map_flat_body<STOCH, PASSES, true>(J, bits, bid == 0, red, key0, key1, first);
        return;
    }
    const uint32_t* __restrict__ x = J.x;
    int8_t* __restrict__ q = J.q;
    int8_t* __restrict__ qT = J.qT;
    const int64_t rows = J.rows, cols = J.cols;
    unsigned rb, cb;
    tile_of_workgroup(J, bid, &rb, &cb);
    const int64_t r0 = static_cast<int64_t>(rb) * TR;
    const int64_t c0 = static_cast<int64_t>(cb) * TC;
    if (r0 + TR <= rows && c0 + TC <= cols)
        map_tile_body<STOCH, false, PASSES, TC>(x, rows, cols, J, bits, bid == 0, red, q, qT, key0, key1, J.sid0, J.sid1, r0, c0, stage, e_true);
    else
        map_tile_body<STOCH, true, PASSES, TC>(x, rows, cols, J, bits, bid == 0, red, q, qT, key0, key1, J.sid0, J.sid1, r0, c0, stage, e_true);
}

// Scale and map in ONE pass over the tensor, for a caller that has a guess of the scale (the tensor's scale of
// the previous training step: the largest exponent of a weight, an activation or a gradient tensor seldom moves
// from one step to the next).  Every workgroup maps its tiles with the guess and keeps the largest magnitude it
// saw; the launch leaves one exponent per workgroup (at most kGuessBlocks: a tile a workgroup up to that many, each a byte)
// and the guess it used.  The launch that follows (k_map_tile with guess_used
// set) computes the true scale from the maxima: equal to the guess - the bytes written here are exactly what the
// two-pass path writes, and that launch ends at once; different, or no usable guess (outside 1 .. 255) - it
// maps the tensor again with the true scale.  4 B read + 2 B written per element instead of 8 + 2 on a hit.
template <bool STOCH, int PASSES, int TC>
__global__ __launch_bounds__(kMapThreads) void k_map_tile_guess(const MapJobs jobs, uint32_t key0, uint32_t key1, int bits) {
    constexpr int RGP = kMapThreads / (TC / 4);
    constexpr int TR = 4 * RGP * PASSES;
    __shared__ uint32_t stage[TC * (RGP * PASSES + 1)];
    __shared__ uint32_t red[kMapThreads / 64];
    const bool second = blockIdx.x >= static_cast<unsigned>(jobs.j[0].guess_blocks);       // workgroup-uniform
    const MapJob& J = jobs.j[second ? 1 : 0];
    const unsigned first = blockIdx.x - (second ? jobs.j[0].guess_blocks : 0), step = J.guess_blocks;
    int guess = J.e_guess[0];
    if (guess < 1 || guess > 255) guess = 0;
    if (first == 0 && threadIdx.x == 0) J.guess_used[0] = guess;
    uint32_t seen = 0;
#pragma unroll 1
    for (unsigned tile = first; tile < J.blocks; tile += step) {
        if (tile != first) __syncthreads();      // the staging area is read by other threads than those that fill it for the next tile
        unsigned rb, cb;
        tile_of_workgroup(J, tile, &rb, &cb);
        const int64_t r0 = static_cast<int64_t>(rb) * TR;
        const int64_t c0 = static_cast<int64_t>(cb) * TC;
        if (r0 + TR <= J.rows && c0 + TC <= J.cols)
            map_tile_body<STOCH, false, PASSES, TC, true>(J.x, J.rows, J.cols, J, bits, false, red, J.q, J.qT, key0, key1, J.sid0,
                                                          J.sid1, r0, c0, stage, guess, guess != 0, &seen);
        else
            map_tile_body<STOCH, true, PASSES, TC, true>(J.x, J.rows, J.cols, J, bits, false, red, J.q, J.qT, key0, key1, J.sid0,
                                                         J.sid1, r0, c0, stage, guess, guess != 0, &seen);
    }
    seen = block_max(seen, red);
    if (threadIdx.x == 0) J.guess_maxima[first] = static_cast<uint8_t>(seen >> 23);
}

// One element per thread, any shape and alignment.
template <bool STOCH>
__global__ __launch_bounds__(kMapThreads) void k_map_generic(const uint32_t* __restrict__ x, int64_t rows, int64_t cols,
                                                             const int32_t* __restrict__ e_in,
                                                             const uint32_t* __restrict__ partials, int n_partials,
                                                             int32_t* __restrict__ e_out, int8_t* __restrict__ q,
                                                             int8_t* __restrict__ qT, uint32_t key0, uint32_t key1,
                                                             uint32_t sid0, uint32_t sid1, int bits) {
    __shared__ uint32_t red[kMapThreads / 64];
    const MapCfg cfg = make_cfg(resolve_scale(e_in, partials, partials_share(partials, n_partials), e_out, red, blockIdx.x == 0), bits);
    const uint64_t n = static_cast<uint64_t>(rows) * static_cast<uint64_t>(cols);
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kMapThreads + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * kMapThreads) {
        const uint32_t b = x[i];
        uint32_t word = 0;
        if (STOCH) {
            const uint64_t blk = i >> 2;
            const uint4 w = philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(blk >> 32), sid0, sid1, key0, key1);
            const uint32_t sel = static_cast<uint32_t>(i & 3u);
            word = sel == 0 ? w.x : sel == 1 ? w.y : sel == 2 ? w.z : w.w;
        }
        const int8_t v = static_cast<int8_t>(with_sign(magnitude_full<STOCH>(b, word, cfg), b));
        if (q) q[i] = v;
        if (qT) {
            const uint64_t r = i / static_cast<uint64_t>(cols), c = i % static_cast<uint64_t>(cols);
            qT[c * static_cast<uint64_t>(rows) + r] = v;
        }
    }
}

static MapPlan plan_map(const MapTensor& t) {
    return plan_map(t.rows, t.cols, aligned(t.x, 16) && aligned(t.q, 16) && aligned(t.qT, 16), t.qT != nullptr);
}

static MapJob make_job(const MapTensor& t, int tc, int passes, bool flat) {
    MapJob j;
    const int64_t tr = (tc == 128 ? 128 : 256) / 4 * passes;
    j.x = reinterpret_cast<const uint32_t*>(t.x);
    j.rows = t.rows;
    j.cols = t.cols;
    j.e_in = t.e_in;
    j.partials = t.partials;
    j.n_partials = t.n_partials;
    j.e_out = t.e_out;
    j.q = t.q;
    j.qT = t.qT;
    j.sid0 = static_cast<uint32_t>(t.stream_id);
    j.sid1 = static_cast<uint32_t>(t.stream_id >> 32);
    j.flat = flat ? 1 : 0;
    j.tiles_c = flat ? 1 : static_cast<int>((t.cols + tc - 1) / tc);
    j.blocks = static_cast<unsigned>(flat ? (t.rows * t.cols + kFlatTileElements * passes - 1) / (kFlatTileElements * passes)
                                          : ((t.rows + tr - 1) / tr) * j.tiles_c);
    const bool shared_lines = j.tiles_c > 1 && t.cols % 128 != 0;
    j.xcd_blocks = shared_lines ? static_cast<unsigned>((t.rows + tr - 1) / tr / 8 * 8 * j.tiles_c) : 0u;
    j.e_guess = nullptr;
    j.guess_maxima = nullptr;
    j.guess_blocks = 0;
    j.guess_used = nullptr;
    return j;
}

static void launch_tiles(const MapJobs& jobs, int tc, int passes, bool stoch, uint32_t k0, uint32_t k1, int bits,
                         hipStream_t s) {
    const dim3 grid(jobs.j[0].blocks + jobs.j[1].blocks), block(kMapThreads);
    const bool flat = jobs.j[0].flat || (jobs.j[1].blocks != 0 && jobs.j[1].flat);
#define FXP_MAP_LAUNCH(STOCH, PASSES, TC)                                                                          \
    do {                                                                                                           \
        auto kernel = flat ? k_map_tile<STOCH, PASSES, TC, true> : k_map_tile<STOCH, PASSES, TC, false>;            \
        hipLaunchKernelGGL(kernel, grid, block, 0, s, jobs, k0, k1, bits);                                          \
    } while (0)
#define FXP_MAP_PICK(TC)                                   \
    if (stoch) {                                           \
        if (passes == 4) FXP_MAP_LAUNCH(true, 4, TC);      \
        else if (passes == 2) FXP_MAP_LAUNCH(true, 2, TC); \
        else FXP_MAP_LAUNCH(true, 1, TC);                  \
    } else {                                               \
        if (passes == 4) FXP_MAP_LAUNCH(false, 4, TC);     \
        else if (passes == 2) FXP_MAP_LAUNCH(false, 2, TC);\
        else FXP_MAP_LAUNCH(false, 1, TC);                 \
    }
    if (tc == 128) { FXP_MAP_PICK(128); }
    else { FXP_MAP_PICK(64); }
#undef FXP_MAP_PICK
#undef FXP_MAP_LAUNCH
}

static void launch_tiles_guess(const MapJobs& jobs, unsigned grid_x, int tc, int passes, bool stoch, uint32_t k0, uint32_t k1,
                               int bits, hipStream_t s) {
    const dim3 grid(grid_x), block(kMapThreads);
#define FXP_MAP_LAUNCH(STOCH, PASSES, TC) \
    hipLaunchKernelGGL((k_map_tile_guess<STOCH, PASSES, TC>), grid, block, 0, s, jobs, k0, k1, bits)
#define FXP_MAP_PICK(TC)                                   \
    if (stoch) {                                           \
        if (passes == 4) FXP_MAP_LAUNCH(true, 4, TC);      \
        else if (passes == 2) FXP_MAP_LAUNCH(true, 2, TC); \
        else FXP_MAP_LAUNCH(true, 1, TC);                  \
    } else {                                               \
        if (passes == 4) FXP_MAP_LAUNCH(false, 4, TC);     \
        else if (passes == 2) FXP_MAP_LAUNCH(false, 2, TC);\
        else FXP_MAP_LAUNCH(false, 1, TC);                 \
    }
    if (tc == 128) { FXP_MAP_PICK(128); }
    else { FXP_MAP_PICK(64); }
#undef FXP_MAP_PICK
#undef FXP_MAP_LAUNCH
}

// Scale + map of one or two tensors (b may be null) with the scales their e_out words hold on entry taken as
// guesses: one pass over the tensors and a launch that verifies (and repairs, should a guess be off).  area_a /
// area_b: kMaxPartials words of scratch each.  Returns kNoGuessPath when the tensors do not take the tiled
// kernel together or are too small for the guess to pay (the caller then takes the two-pass path).
int scale_map_guess_launch(const MapTensor& a, const MapTensor* b, uint32_t* area_a, uint32_t* area_b, uint64_t seed,
                           int rounding, int bits, hipStream_t s) {
    const MapPlan pa = plan_map(a);
    const MapPlan pb = b ? plan_map(*b) : pa;
    const int64_t na = a.rows * a.cols, nb = b ? b->rows * b->cols : 0;
    // below a few million elements a scale reduction costs what the verifying launch costs
    if (std::max(na, nb) < kGuessMinElements) return kNoGuessPath;
    // (tiles, whether or not an ordinary map would take the tensor flat)
    if (!pa.tiles || !pb.tiles || pa.any || pb.any) return kNoGuessPath;
    if (pa.tc != pb.tc) return kGuessOneByOne;        // different tile widths: no common launch, but each may guess alone
    int passes = na >= nb ? pa.passes : pb.passes;
    // The body that also keeps the maximum holds 111 registers for two passes and 143 for four: two, where every workgroup then
    // still has one tile (12608 x 2304 34.8 us for 36.4; 8192 x 8192, three tiles of two passes for two of four, step 1612 for 1600).
    if (passes == 4 && std::max(make_job(a, pa.tc, 2, false).blocks, b ? make_job(*b, pa.tc, 2, false).blocks : 0u) <= kGuessBlocks) passes = 2;
    MapJobs jobs;
    jobs.j[0] = make_job(a, pa.tc, passes, false);
    if (b) jobs.j[1] = make_job(*b, pa.tc, passes, false);
    else { jobs.j[1] = jobs.j[0]; jobs.j[1].blocks = 0; }
    const uint64_t total = static_cast<uint64_t>(jobs.j[0].blocks) + jobs.j[1].blocks;
    if (total >= (uint64_t{1} << 31)) return kNoGuessPath;
    unsigned grid = 0;
    uint32_t* areas[2] = {area_a, area_b};
    const MapTensor* ts[2] = {&a, b};
    for (int j = 0; j < 2; ++j) {
        if (jobs.j[j].blocks == 0) continue;
        jobs.j[j].e_guess = ts[j]->e_out;                                   // last step's scale, if the caller kept it
        jobs.j[j].guess_maxima = reinterpret_cast<uint8_t*>(areas[j]);
        const unsigned per = (jobs.j[j].blocks + kGuessBlocks - 1) / kGuessBlocks;       // tiles of a workgroup
        jobs.j[j].guess_blocks = static_cast<int>((jobs.j[j].blocks + per - 1) / per);
        grid += jobs.j[j].guess_blocks;
        jobs.j[j].guess_used = reinterpret_cast<int32_t*>(areas[j] + kGuessBlocks / 4);
        jobs.j[j].e_in = nullptr;
        jobs.j[j].partials = nullptr;
    }
    const bool stoch = rounding == FXP_ROUND_STOCHASTIC;
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    launch_tiles_guess(jobs, grid, pa.tc, passes, stoch, k0, k1, bits, s);
    int rc = launch_status();
    if (rc) return rc;
    // the launch that verifies: an ordinary map launch whose workgroups look at the maxima first
    launch_tiles(jobs, pa.tc, passes, stoch, k0, k1, bits, s);
    return launch_status();
}

int map_launch(const MapTensor& t, uint64_t seed, int rounding, int bits, hipStream_t s) {
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    const bool stoch = rounding == FXP_ROUND_STOCHASTIC;
    const MapPlan p = plan_map(t);
    if (p.tile_path && p.any && !p.flat) return map_rows_launch(t, nullptr, seed, rounding, bits, s);
    if (p.tile_path) {
        MapJobs jobs;
        jobs.j[0] = make_job(t, p.tc, p.passes, p.flat);
        jobs.j[1] = jobs.j[0];
        jobs.j[1].blocks = 0;
        launch_tiles(jobs, p.tc, p.passes, stoch, k0, k1, bits, s);
    } else {
        const uint32_t s0 = static_cast<uint32_t>(t.stream_id), s1 = static_cast<uint32_t>(t.stream_id >> 32);
        const uint32_t* xb = reinterpret_cast<const uint32_t*>(t.x);
        const uint64_t n = static_cast<uint64_t>(t.rows) * static_cast<uint64_t>(t.cols);
        uint64_t want = (n + kMapThreads - 1) / kMapThreads;
        const dim3 grid(static_cast<unsigned>(want < 1 ? 1 : (want > 16384 ? 16384 : want))), block(kMapThreads);
        if (stoch)
            hipLaunchKernelGGL(k_map_generic<true>, grid, block, 0, s, xb, t.rows, t.cols, t.e_in, t.partials, t.n_partials,
                               t.e_out, t.q, t.qT, k0, k1, s0, s1, bits);
        else
            hipLaunchKernelGGL(k_map_generic<false>, grid, block, 0, s, xb, t.rows, t.cols, t.e_in, t.partials, t.n_partials,
                               t.e_out, t.q, t.qT, k0, k1, s0, s1, bits);
    }
    return launch_status();
}

// Two tensors in one launch when both are tiled or flat; the tile height is the one the larger tensor would pick.  Otherwise one
// launch each.
int map_launch2(const MapTensor& a, const MapTensor& b, uint64_t seed, int rounding, int bits, hipStream_t s) {
    MapPlan pa = plan_map(a), pb = plan_map(b);
    if (tiles_for_both(pa, a.cols, pb, b.cols)) {
        pa = plan_map(a.rows, a.cols, true, true);
        pb = plan_map(b.rows, b.cols, true, true);
    }
    // tiles of quads for both if one needs them, or if their tile widths differ (attention steps, in two launches / one: 24 x 80 x 64
    // 63.4 / 60.8 us, 768 x 208 x 64 381.5 / 379.4, 576 x 256 x 64 366.7 / 361.4)
    const bool rows = (pa.any && !pa.flat) || (pb.any && !pb.flat) || (pa.tc != pb.tc && !pa.flat && !pb.flat);
    if (pa.tile_path && pb.tile_path && rows) return map_rows_launch(a, &b, seed, rounding, bits, s);
    if (!pa.tile_path || !pb.tile_path) {
        const int rc = map_launch(a, seed, rounding, bits, s);
        return rc ? rc : map_launch(b, seed, rounding, bits, s);
    }
    const int passes = a.rows * a.cols >= b.rows * b.cols ? pa.passes : pb.passes;
    const int tc = pa.flat ? pb.tc : pa.tc;          // a flat tensor has no tile width of its own
    MapJobs jobs;
    jobs.j[0] = make_job(a, tc, passes, pa.flat);
    jobs.j[1] = make_job(b, tc, passes, pb.flat);
    if (static_cast<uint64_t>(jobs.j[0].blocks) + jobs.j[1].blocks >= (uint64_t{1} << 31)) {
        const int rc = map_launch(a, seed, rounding, bits, s);
        return rc ? rc : map_launch(b, seed, rounding, bits, s);
    }
    launch_tiles(jobs, tc, passes, rounding == FXP_ROUND_STOCHASTIC, static_cast<uint32_t>(seed),
                 static_cast<uint32_t>(seed >> 32), bits, s);
    return launch_status();
}

static int check_map_args(const float* x, int64_t rows, int64_t cols, const void* e, int8_t* q, int8_t* qT, int rounding,
                          int bits) {
    if (rows < 0 || cols < 0) return FXP_ERR_DIMS;
    if (rows > 0 && cols > 0 && rows > (int64_t{1} << 62) / cols) return FXP_ERR_DIMS;
    if (!e || (!q && !qT) || (rows * cols > 0 && !x)) return FXP_ERR_NULL;
    if (rounding != FXP_ROUND_STOCHASTIC && rounding != FXP_ROUND_NEAREST) return FXP_ERR_ROUNDING;
    if (bits < 2 || bits > 8) return FXP_ERR_BITS;
    if (!aligned(x, 4) || !aligned(e, 4)) return FXP_ERR_ALIGN;
    return FXP_OK;
}

}  // namespace fxp

extern "C" int fxp_map(const float* x, int64_t rows, int64_t cols, const int32_t* e_max, int8_t* q, int8_t* qT,
                       uint64_t seed, uint64_t stream_id, int rounding, int bits, void* stream) {
    int rc = fxp::check_map_args(x, rows, cols, e_max, q, qT, rounding, bits);
    if (rc) return rc;
    if (rows * cols == 0) return FXP_OK;
    fxp::MapTensor t{x, rows, cols, e_max, nullptr, 0, nullptr, q, qT, stream_id};
    return fxp::map_launch(t, seed, rounding, bits, static_cast<hipStream_t>(stream));
}

extern "C" int fxp_map_absmax(const float* x, int64_t rows, int64_t cols, const uint32_t* absmax, int32_t* e_max, int8_t* q,
                              int8_t* qT, uint64_t seed, uint64_t stream_id, int rounding, int bits, void* stream) {
    int rc = fxp::check_map_args(x, rows, cols, e_max, q, qT, rounding, bits);
    if (rc) return rc;
    if (!absmax) return FXP_ERR_NULL;
    if (!fxp::aligned(absmax, 4)) return FXP_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (rows * cols == 0) return fxp::scale_finish(absmax, FXP_ABSMAX_WORDS, e_max, s);     // only the scale
    // the words are a list of block maxima: the map kernel turns them into the scale and publishes it
    const fxp::MapTensor t{x, rows, cols, nullptr, absmax, FXP_ABSMAX_WORDS, e_max, q, qT, stream_id};
    return fxp::map_launch(t, seed, rounding, bits, s);
}

extern "C" int fxp_scale_map(const float* x, int64_t rows, int64_t cols, int32_t* e_max, int8_t* q, int8_t* qT,
                             uint64_t seed, uint64_t stream_id, int rounding, int bits, void* ws, size_t ws_bytes,
                             void* stream) {
    int rc = fxp::check_map_args(x, rows, cols, e_max, q, qT, rounding, bits);
    if (rc) return rc;
    if (!ws || ws_bytes < fxp::kScaleWsBytes) return FXP_ERR_WORKSPACE;
    if (!fxp::aligned(ws, 4)) return FXP_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint32_t* partials = static_cast<uint32_t*>(ws);
    if (rows * cols == 0) {
        int np = 0;
        rc = fxp::scale_partials(x, 0, partials, &np, s);
        return rc ? rc : fxp::scale_finish(partials, np, e_max, s);
    }
    return fxp::scale_and_map(x, rows, cols, e_max, q, qT, seed, stream_id, rounding, bits, partials, s);
}

static int check_desc(const fxp_map_desc* d, int rounding, int bits) {
    if (!d) return FXP_ERR_NULL;
    return fxp::check_map_args(d->x, d->rows, d->cols, d->e_max, d->q, d->qT, rounding, bits);
}

extern "C" int fxp_map2(const fxp_map_desc* a, const fxp_map_desc* b, uint64_t seed, int rounding, int bits, void* stream) {
    int rc = check_desc(a, rounding, bits);
    if (!rc) rc = check_desc(b, rounding, bits);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const fxp::MapTensor ta{a->x, a->rows, a->cols, a->e_max, nullptr, 0, nullptr, a->q, a->qT, a->stream_id};
    const fxp::MapTensor tb{b->x, b->rows, b->cols, b->e_max, nullptr, 0, nullptr, b->q, b->qT, b->stream_id};
    if (a->rows * a->cols == 0 || b->rows * b->cols == 0) {     // an empty tensor has nothing to launch
        if (a->rows * a->cols && (rc = fxp::map_launch(ta, seed, rounding, bits, s))) return rc;
        if (b->rows * b->cols && (rc = fxp::map_launch(tb, seed, rounding, bits, s))) return rc;
        return FXP_OK;
    }
    return fxp::map_launch2(ta, tb, seed, rounding, bits, s);
}

extern "C" int fxp_scale_map2(const fxp_map_desc* a, const fxp_map_desc* b, uint64_t seed, int rounding, int bits, void* ws,
                              size_t ws_bytes, void* stream) {
    int rc = check_desc(a, rounding, bits);
    if (!rc) rc = check_desc(b, rounding, bits);
    if (rc) return rc;
    if (!ws || ws_bytes < 2 * fxp::kScaleWsBytes) return FXP_ERR_WORKSPACE;
    if (!fxp::aligned(ws, 4)) return FXP_ERR_ALIGN;
    uint32_t* pa = static_cast<uint32_t*>(ws);
    uint32_t* pb = pa + fxp::kMaxPartials;
    if (a->rows * a->cols == 0 || b->rows * b->cols == 0) {     // an empty tensor: the single-tensor path, twice
        rc = fxp_scale_map(a->x, a->rows, a->cols, a->e_max, a->q, a->qT, seed, a->stream_id, rounding, bits, pa,
                           fxp::kScaleWsBytes, stream);
        return rc ? rc
                  : fxp_scale_map(b->x, b->rows, b->cols, b->e_max, b->q, b->qT, seed, b->stream_id, rounding, bits, pb,
                                  fxp::kScaleWsBytes, stream);
    }
    const fxp::MapTensor ta{a->x, a->rows, a->cols, nullptr, pa, 0, a->e_max, a->q, a->qT, a->stream_id};
    const fxp::MapTensor tb{b->x, b->rows, b->cols, nullptr, pb, 0, b->e_max, b->q, b->qT, b->stream_id};
    return fxp::scale_and_map2(ta, tb, seed, rounding, bits, static_cast<hipStream_t>(stream));
}
