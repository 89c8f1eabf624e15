// Mapping (see fxp_map.hip for what is computed) of tensors whose rows are not whole quads or that lie off the 16-byte grid,
// and of small tensors, whose scale is worked out in the same launch.
//
// The random words belong to quads of consecutive elements (element i: word i mod 4 of block i / 4) and the bytes of a
// row-major tensor lie in element order, so a thread takes one such quad, whatever row it starts in: one 16-byte load, one
// Philox block, one dword of the row-major copy.  A window of w columns meets at most (w + 6) / 4 quads of a row; those at
// its ends reach into the neighbouring windows, and the window a quad begins in writes its dword.  For the transposed copy the
// bytes go to LDS one by one, [column][row] with room for three columns on either side, and leave it as 16-byte pieces along
// the rows of qT.
// (18912 x 197, both copies, 18.6 MB read and written: 14.8 us as tiles of 4 x 4 elements, which need five blocks of random
// words per 16 elements and element-wise loads at their edges.  Those were ahead in one place: tall tensors of 64 or 128 columns
// whose base is off the grid, which they cut into whole tiles with longer runs of qT - 262144 x 64 27.7 / 30.8 us to nearest and
// 30.5 / 33.0, 65536 x 128 16.7 / 18.0 and 19.5 / 20.3; 96 columns 68.1 / 55.1, 192 59.1 / 55.3.)
#include <algorithm>

#include "fxp_internal.h"
#include "fxp_map_device.h"
#include "fxp_map_plan.h"

namespace fxp {

struct RowsJob {
    const uint32_t* x;
    int64_t rows, cols;
    const int32_t* e_in;
    const uint32_t* partials;
    int n_partials;
    int32_t* e_out;
    int8_t* q;
    int8_t* qT;
    uint32_t sid0, sid1;
    uint32_t width, quads, magic;    // columns of a window, quads of a row of it, ceil(2^32 / quads)
    uint32_t inner;                  // tiles that follow each other: the windows of a row block, or (down) the row blocks of a window
    int down;
    unsigned blocks;
    int flat;                        // row-major copy only (map_flat_body)
};
struct RowsJobs {
    RowsJob j[2];
};

// Workgroup bid of `blocks` works on tile number ...: one run of tiles per XCD, so that the lines which neighbouring windows
// (and, in the transposed copy, neighbouring row blocks) share are met in one L2.  Of up to eight row blocks, whose tiles of one window
// write lines of the transposed copy between them, these are neighbours; else the windows of a row block (1000 x 50257 75.7 -> 67.3 us,
// 64 x 50257 7.5 -> 7.2, rounding to nearest 6.0 -> 5.6).
__device__ inline unsigned tile_in_xcd_run(unsigned bid, unsigned blocks) {
    const unsigned per = blocks / 8u, more = blocks % 8u, xcd = bid % 8u, at = bid / 8u;
    return xcd < more ? xcd * (per + 1) + at : more * (per + 1) + (xcd - more) * per + at;
}

// Largest magnitude bits of a whole tensor, by every workgroup for itself, bound by what a CU reads from L2: in chunks of sixteen
// 16-byte loads a thread, each workgroup from a chunk of its own on so that not all of them miss the same lines at once, and eight
// for a rest of half a chunk or less (256 x 448 6.8 -> 6.4 us).  The compiler keeps nine to ten in flight; all sixteen, held together
// by a scheduling barrier, are slower (256 x 256 4.9 -> 5.1, 256 x 384 5.8 -> 6.2).
constexpr int kScanThreads = 512;
__device__ inline uint32_t scan_absmax(const uint32_t* __restrict__ x, uint32_t n, unsigned bid) {
    const uint32_t kAbs = 0x7fffffffu;
    const uint32_t mis = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(x) >> 2) & 3u;
    const uint32_t head = min(mis ? 4 - mis : 0u, n), nvec = (n - head) >> 2, tail0 = head + 4 * nvec;
    const uint4* xv = reinterpret_cast<const uint4*>(x + head);
    uint32_t m = 0;
    if (threadIdx.x < head) m = x[threadIdx.x] & kAbs;
    if (tail0 + threadIdx.x < n) m = max(m, x[tail0 + threadIdx.x] & kAbs);       // fewer than four
    auto chunk = [&](uint32_t first, auto loads) {
        constexpr uint32_t kLoads = decltype(loads)::value;
        uint4 v[kLoads];
#pragma unroll
        for (uint32_t k = 0; k < kLoads; ++k) v[k] = xv[min(first + k * kScanThreads + threadIdx.x, nvec - 1)];
#pragma unroll
        for (uint32_t k = 0; k < kLoads; ++k) m = max(m, absmax4(v[k]));
    };
    constexpr uint32_t kChunk = 16 * kScanThreads;
    if (nvec == 0) return m;
    const uint32_t chunks = (nvec + kChunk / 2 - 1) / kChunk;                    // and half of one, or less
    uint32_t at = chunks ? bid % chunks : 0;
    for (uint32_t c = 0; c < chunks; ++c) {
        chunk(at * kChunk, std::integral_constant<uint32_t, 16>{});
        if (++at == chunks) at = 0;
    }
    if (nvec > chunks * kChunk) chunk(chunks * kChunk, std::integral_constant<uint32_t, 8>{});
    return m;
}

// One tile: TR rows x J.width columns.  SCAN: the scale is not given and has no block maxima, see scan_absmax.
// The elements of the tensor's last, short quad (n % 4 != 0) are mapped one by one.  All per-thread addressing is a 32-bit element
// offset from the quad that the tile's first element lies in.
template <bool STOCH, int TR, bool SCAN>
__device__ inline void map_rows_body(const RowsJob& J, int bits, uint32_t key0, uint32_t key1, unsigned bid, uint32_t* red,
                                     uint8_t* stage) {
    constexpr int TS = TR + 4;                    // bytes per staged column: an odd number of dwords
    constexpr int NT = SCAN ? kScanThreads : kMapThreads;
    constexpr int U = SCAN ? 1 : 4;               // quads in flight per thread
    constexpr uint32_t kOff = 0xffffffffu;        // offset of a lane without a quad
    const unsigned tile = tile_in_xcd_run(bid, J.blocks), outer = tile / J.inner, inner = tile - outer * J.inner;
    const unsigned rb = J.down ? inner : outer, cb = J.down ? outer : inner;
    const int64_t r0 = static_cast<int64_t>(rb) * TR;
    const uint32_t c0 = cb * J.width, ucols = static_cast<uint32_t>(J.cols);
    const uint32_t rows_here = static_cast<uint32_t>(min<int64_t>(TR, J.rows - r0));
    const int w_here = static_cast<int>(min(J.width, ucols - c0));
    const uint64_t n = static_cast<uint64_t>(J.rows) * ucols, origin = static_cast<uint64_t>(r0) * ucols + c0;
    const uint32_t lead0 = static_cast<uint32_t>(origin) & 3u;
    const uint32_t* __restrict__ x = J.x + (origin - lead0);
    int8_t* __restrict__ q = J.q ? J.q + (origin - lead0) : nullptr;
    int8_t* __restrict__ qT = J.qT;
    const uint64_t blk0 = origin >> 2;
    // quads from `whole` on are not all inside the tensor
    const uint64_t n4 = n & ~uint64_t{3};
    const uint32_t whole = n4 > origin - lead0 ? static_cast<uint32_t>(min<uint64_t>(n4 - (origin - lead0), kOff)) : 0u;
    const uint32_t total = whole ? rows_here * J.quads : 0u;
    struct Quads {
        uint4 v[U];
        uint32_t rel[U];                          // element offset of the quad, kOff: none
        int lds[U];                               // where its first element is staged; columns -3 .. w + 2 have room there
    };
    auto load = [&](uint32_t id, Quads& a) {
#pragma unroll
        for (int u = 0; u < U; ++u, id += NT) {
            const uint32_t row = __umulhi(id, J.magic), off = lead0 + row * ucols;
            const uint32_t rel = (off & ~3u) + 4 * (id - row * J.quads);
            const int col = static_cast<int>(rel - off);
            const bool on = id < total && col < w_here && rel < whole;
            a.rel[u] = on ? rel : kOff;
            a.lds[u] = (col + 3) * TS + static_cast<int>(row);
            a.v[u] = load_quad(reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(x) + (on ? 4 * rel : 0u)));
        }
    };
    Quads cur, nxt;
    uint32_t id = threadIdx.x;
    const uint32_t share = SCAN ? 0u : partials_share(J.partials, J.n_partials);
    if (total) load(id, cur);                     // (without the branch, and its wait for these before the scale: up to 7 % slower)
    int e;
    if constexpr (SCAN) {
        const uint32_t m = block_max<kScanThreads / 64>(scan_absmax(J.x, static_cast<uint32_t>(n), bid), red);
        e = max(1, static_cast<int>(m >> 23));
        if (bid == 0 && threadIdx.x == 0) J.e_out[0] = e;
    } else {
        e = resolve_scale(J.e_in, J.partials, share, J.e_out, red, bid == 0);
    }
    const MapCfg cfg = make_cfg(e, bits);
    const bool scale_ok = cfg.e_max >= 25 && cfg.e_max < 255;
    const uint32_t rounds = (total + U * NT - 1) / (U * NT);
    for (uint32_t round = 0; round < rounds; ++round) {
        if (round + 1 < rounds) load(id += U * NT, nxt);
        uint32_t o[U], q_or = 0;
        uint64_t bad = 0;                          // wave-uniform: any lane with an uncovered element
        auto words_of = [&](int u) {
            const uint64_t blk = blk0 + (cur.rel[u] >> 2);
            return STOCH ? philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(blk >> 32), J.sid0, J.sid1, key0, key1)
                         : make_uint4(0, 0, 0, 0);
        };
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = map_quad_fast<STOCH>(cur.v[u], words_of(u), cfg, q_or, bad);
        if (!scale_ok || bad != 0 || (q_or & ~cfg.sat)) {
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = map_quad_full<STOCH>(cur.v[u], words_of(u), cfg);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (cur.rel[u] == kOff) continue;
            // (it begins in this window: column 0 or beyond)
            if (q != nullptr && cur.lds[u] >= 3 * TS) reinterpret_cast<Bytes4*>(q + cur.rel[u])->x = o[u];
            if (qT != nullptr) {
#pragma unroll
                for (int k = 0; k < 4; ++k) stage[cur.lds[u] + k * TS] = static_cast<uint8_t>(o[u] >> (8 * k));
            }
        }
        cur = nxt;
    }
    if ((n & 3u) != 0 && r0 + TR >= J.rows && threadIdx.x < (n & 3u)) {
        const uint64_t i = n4 + threadIdx.x;
        const int col = static_cast<int>(static_cast<int64_t>(i) - (J.rows - 1) * J.cols - c0);
        if (col >= 0 && col < w_here) {
            const uint4 w = STOCH ? philox4x32_10(static_cast<uint32_t>(n4 >> 2), static_cast<uint32_t>(n4 >> 34), J.sid0, J.sid1, key0, key1)
                                  : make_uint4(0, 0, 0, 0);
            const uint32_t b = J.x[i];
            const uint32_t v = with_sign(magnitude_full<STOCH>(b, threadIdx.x == 0 ? w.x : threadIdx.x == 1 ? w.y : w.z, cfg), b);
            if (J.q != nullptr) J.q[i] = static_cast<int8_t>(v);
            stage[(col + 3) * TS + rows_here - 1] = static_cast<uint8_t>(v);
        }
    }
    if (qT == nullptr) return;
    __syncthreads();
    int8_t* qTt = qT + static_cast<uint64_t>(c0) * J.rows + r0;
    constexpr uint32_t PIECES = TR / 16;
    for (uint32_t p = threadIdx.x; p < static_cast<uint32_t>(w_here) * PIECES; p += NT) {
        const uint32_t c = p / PIECES, ch = p % PIECES;
        if (16 * ch >= rows_here) continue;
        const uint32_t* src = reinterpret_cast<const uint32_t*>(stage + (c + 3) * TS) + 4 * ch;
        int8_t* dst = qTt + static_cast<uint64_t>(c) * J.rows + 16 * ch;
        if (16 * ch + 16 <= rows_here) {
            *reinterpret_cast<Bytes16*>(dst) = Bytes16{src[0], src[1], src[2], src[3]};
        } else {
            for (uint32_t r = 0; 16 * ch + r < rows_here; ++r) dst[r] = static_cast<int8_t>(src[r >> 2] >> (8 * (r & 3)));
        }
    }
}

// Five waves per SIMD (96 registers) where that spills nothing: 98 leave four (49344 x 257 18.8 -> 17.8 us, 25000 x 301 13.9 -> 13.3,
// 18912 x 197 8.4 -> 8.2; 8191 x 8191, bound by memory, 97 -> 100).
template <bool STOCH, int TR, bool SCAN, bool FLAT>
__global__ __launch_bounds__(SCAN ? kScanThreads : kMapThreads, SCAN ? 1 : FLAT ? 4 : 5) void k_map_rows(const RowsJobs jobs, uint32_t key0, uint32_t key1, int bits) {
    __shared__ __align__(16) uint8_t stage[(kRowsWidth + 6) * (TR + 4)];
    __shared__ uint32_t red[kScanThreads / 64];
    const bool second = blockIdx.x >= jobs.j[0].blocks;            // workgroup-uniform
    const RowsJob& J = jobs.j[second ? 1 : 0];
    const unsigned bid = blockIdx.x - (second ? jobs.j[0].blocks : 0u);
    if (FLAT && J.flat) {
        constexpr int PASSES = TR / 32;
        const uint64_t first = static_cast<uint64_t>(bid) * (4 * kMapThreads * PASSES);
        const uint64_t whole = static_cast<uint64_t>(J.rows) * static_cast<uint64_t>(J.cols) >> 2;
        if (first + 4 * kMapThreads * PASSES <= whole) map_flat_body<STOCH, PASSES, false>(J, bits, bid == 0, red, key0, key1, first);
        else map_flat_body<STOCH, PASSES, true>(J, bits, bid == 0, red, key0, key1, first);
        return;
    }
    map_rows_body<STOCH, TR, SCAN>(J, bits, key0, key1, bid, red, stage);
}

static RowsJob make_rows_job(const MapTensor& t, const RowsPlan& p, bool flat) {
    RowsJob j;
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
    j.width = p.width;
    j.quads = p.quads;
    j.magic = p.magic;
    const int64_t high = p.blocks / p.windows;
    j.down = high <= 8 ? 1 : 0;
    j.inner = j.down ? static_cast<uint32_t>(high) : p.windows;
    j.flat = flat ? 1 : 0;
    j.blocks = static_cast<unsigned>(flat ? (t.rows * t.cols + kFlatTileElements * p.tr / 32 - 1) / (kFlatTileElements * p.tr / 32)
                                          : p.blocks);
    return j;
}

static int launch_rows(const RowsJobs& jobs, int tr, bool scan, uint64_t seed, int rounding, int bits, hipStream_t s) {
    const dim3 grid(jobs.j[0].blocks + jobs.j[1].blocks), block(scan ? kScanThreads : kMapThreads);
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    const bool flat = jobs.j[0].flat || jobs.j[1].flat, stoch = rounding == FXP_ROUND_STOCHASTIC;
    auto pick = [&](auto st) {
        constexpr bool S = decltype(st)::value;
        if (scan) return k_map_rows<S, 32, true, false>;
        if (tr == 128) return flat ? k_map_rows<S, 128, false, true> : k_map_rows<S, 128, false, false>;
        if (tr == 64) return flat ? k_map_rows<S, 64, false, true> : k_map_rows<S, 64, false, false>;
        return flat ? k_map_rows<S, 32, false, true> : k_map_rows<S, 32, false, false>;
    };
    const auto kernel = stoch ? pick(std::true_type{}) : pick(std::false_type{});
    hipLaunchKernelGGL(kernel, grid, block, 0, s, jobs, k0, k1, bits);
    return launch_status();
}

// One tensor or two (b may be null), planned as tiles or flat by plan_map.
int map_rows_launch(const MapTensor& a, const MapTensor* b, uint64_t seed, int rounding, int bits, hipStream_t s) {
    const MapTensor* ts[2] = {&a, b};
    MapPlan plans[2] = {};
    for (int j = 0; j < (b ? 2 : 1); ++j) {
        const MapTensor& t = *ts[j];
        plans[j] = plan_map(t.rows, t.cols, aligned(t.x, 16) && aligned(t.q, 16) && aligned(t.qT, 16), t.qT != nullptr);
    }
    const int larger = b && b->rows * b->cols > a.rows * a.cols ? 1 : 0;
    const int tr = rows_height(plans[larger], ts[larger]->rows, ts[larger]->cols);
    RowsJobs jobs{};
    uint64_t blocks = 0;
    for (int j = 0; j < (b ? 2 : 1); ++j) {
        const MapTensor& t = *ts[j];
        const RowsPlan p = j == larger && !plans[j].flat ? plan_rows(t.rows, t.cols) : plan_rows(t.rows, t.cols, tr, rows_windows(t.cols));
        jobs.j[j] = make_rows_job(t, p, plans[j].flat);
        blocks += jobs.j[j].blocks;
    }
    if (b && blocks >= (uint64_t{1} << 31)) {
        const int rc = map_rows_launch(a, nullptr, seed, rounding, bits, s);
        return rc ? rc : map_rows_launch(*b, nullptr, seed, rounding, bits, s);
    }
    return launch_rows(jobs, tr, false, seed, rounding, bits, s);
}

// Scale and map of one tensor or two (b may be null) in one launch: whether they are small enough, and the launch.
bool scale_map_small_fits(const MapTensor& a, const MapTensor* b) {
    const ScanSize sb{b ? b->rows : 0, b ? b->cols : 0};
    return scan_fits(ScanSize{a.rows, a.cols}, b ? &sb : nullptr);
}

int scale_map_small_launch(const MapTensor& a, const MapTensor* b, uint64_t seed, int rounding, int bits, hipStream_t s) {
    RowsJobs jobs{};
    jobs.j[0] = make_rows_job(a, plan_scan(a.rows, a.cols), false);
    if (b) jobs.j[1] = make_rows_job(*b, plan_scan(b->rows, b->cols), false);
    return launch_rows(jobs, 32, true, seed, rounding, bits, s);
}

}  // namespace fxp
