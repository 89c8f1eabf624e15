// Convolutions of thin images (a few channels: the stem of an image model) read straight from the int8 image.
//
// The patch matrix of such a layer is many times its image (7 x 7, stride 2: twelve times), and with 3 bytes per pixel it
// can neither be written nor read in whole 16-byte pieces: stored patches cost the stem of a ResNet-18 (32 x 224 x 224 x 3
// -> 64) 67 us forward and 2.2 ms transposed.  Here the patches exist in registers only.
//   forward : a lane's MFMA operand is 16 consecutive bytes of one filter row of its output pixel - one unaligned load;
//             every filter row is padded to 32 contraction bytes, the padding multiplied by zero weights.
//   weight gradient : the contraction runs over output pixels, so the operand is 16 neighbouring pixels of one tap.  A
//             workgroup holds its image rows in LDS split into planes (one per channel and column phase of the
//             stride), where those 16 bytes are neighbours: five dwords and four byte alignments.
#include <algorithm>

#include "fxp_internal.h"

namespace fxp {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

struct __attribute__((packed, aligned(1))) AnyBytes16 {
    uint32_t x, y, z, w;
};
__device__ inline v4i load_any16(const int8_t* p) {
    const AnyBytes16 b = *reinterpret_cast<const AnyBytes16*>(p);
    v4i v;
    v[0] = static_cast<int>(b.x); v[1] = static_cast<int>(b.y); v[2] = static_cast<int>(b.z); v[3] = static_cast<int>(b.w);
    return v;
}

// the mask of bytes lo .. hi - 1 of a dword (clamped to 0 .. 4)
__device__ inline uint32_t byte_mask(int lo, int hi) {
    lo = min(max(lo, 0), 4);
    hi = min(max(hi, 0), 4);
    const uint32_t below_hi = hi == 4 ? 0xffffffffu : (1u << (8 * hi)) - 1u;
    const uint32_t below_lo = lo == 4 ? 0xffffffffu : (1u << (8 * lo)) - 1u;
    return below_hi & ~below_lo;
}

// Bytes at .. at + 15 of a tensor of `size` >= 16 bytes for operands whose unwanted bytes are zero: the load itself is
// unconditional (from the nearest 16 bytes that lie inside), so that a wave's loads are all in flight before one is
// waited for; keep() then picks the bytes.
__device__ inline v4i load_near16(const int8_t* base, int64_t at, int64_t size) {
    return load_any16(base + min(max(at, int64_t{0}), size - 16));
}
// The 16 bytes at `at` with only those of the mask kept (the wanted ones: lo .. hi - 1).  A lane at one of the tensor's
// ends, whose load was moved, fetches its bytes one by one.
__device__ inline v4i keep(v4i v, const int8_t* base, int64_t at, int64_t size, int lo, int hi, const uint32_t (&mask)[4]) {
    const bool moved = lo < hi && (at < 0 || at > size - 16);
    if (__builtin_amdgcn_ballot_w64(moved) != 0 && moved) {
        v = v4i{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 16; ++b)
            if (b >= lo && b < hi) v[b >> 2] |= static_cast<int>(static_cast<uint32_t>(static_cast<uint8_t>(base[at + b])) << (8 * (b & 3)));
        return v;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) v[d] = lo < hi ? static_cast<int>(static_cast<uint32_t>(v[d]) & mask[d]) : 0;
    return v;
}

// Y[m][co] = unmap(sum over filter rows kh of patch bytes * weights).  A wave owns tiles of 32 output pixels and all
// 32 * FN output channels; the weights, laid out as MFMA operands, are shared through LDS.  Bound by the output, 103 MB
// of the 113 MB that the 32 x 224 x 224 x 3 -> 64 stem moves: 29 us (3.9 TB/s; 118 with the patch matrix stored and read
// back, 57 with every load waited for before the next).
template <int FN>
__global__ __launch_bounds__(256, FN <= 2 ? 4 : 2) void k_conv_thin_fwd(const int8_t* __restrict__ Xq, const int8_t* __restrict__ Wq,
                                                       float* __restrict__ Y, ConvTaps ct, int KH, uint32_t M, int Cout,
                                                       int64_t x_bytes, const int32_t* __restrict__ eA, int bitsA,
                                                       const int32_t* __restrict__ eB, int bitsB, uint32_t tiles) {
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];   // [kh][fragment][lane] x 16 bytes
    constexpr int kRows = 8;                                       // filter rows in flight
    const int row_bytes = ct.KW * ct.C;                            // <= 32
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    for (int id = threadIdx.x; id < KH * FN * 64; id += 256) {
        const int l = id & 63, f = (id >> 6) % FN, kh = (id >> 6) / FN;
        const int co = 32 * f + (l & 31), k0 = 16 * (l >> 5), n = min(16, row_bytes - k0);
        const int64_t w_bytes = static_cast<int64_t>(Cout) * KH * row_bytes;
        const int64_t at = (static_cast<int64_t>(min(co, Cout - 1)) * KH + kh) * row_bytes + k0;
        uint32_t mask[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) mask[d] = byte_mask(0, n - 4 * d);
        const v4i w = keep(load_near16(Wq, at, w_bytes), Wq, at, w_bytes, 0, co < Cout ? n : 0, mask);
        *reinterpret_cast<v4i*>(lds + id * 16) = w;
    }
    __syncthreads();
    const int E = lsb_exponent(eA[0], bitsA) + lsb_exponent(eB[0], bitsB);
    const bool plain = E >= -126 && E <= 127;
    const float unit = __uint_as_float(static_cast<uint32_t>(plain ? E + 127 : 127) << 23);
    const int image_row = ct.W * ct.C;
    for (uint32_t tile = blockIdx.x * 4 + (threadIdx.x >> 6); tile < tiles; tile += gridDim.x * 4) {
        const uint32_t m0 = tile * 32, m = min(m0 + col, M - 1);
        const uint32_t t = m / static_cast<uint32_t>(ct.Wo), n = t / static_cast<uint32_t>(ct.Ho);
        const int h0 = static_cast<int>(t - n * ct.Ho) * ct.stride - ct.pad;
        const int off = (static_cast<int>(m - t * ct.Wo) * ct.stride - ct.padw) * ct.C + 16 * half;   // in the image row
        // bytes of the piece inside the image row and inside the filter row
        const int lo = max(0, -off), hi = min(min(16, image_row - off), row_bytes - 16 * half);
        uint32_t mask[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) mask[d] = byte_mask(lo - 4 * d, hi - 4 * d);
        const int64_t first = static_cast<int64_t>(n) * ct.H * image_row + off;
        v16i acc[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] = 0;
        for (int kb = 0; kb < KH; kb += kRows) {
            v4i a[kRows];
#pragma unroll
            for (int k = 0; k < kRows; ++k)
                if (kb + k < KH) a[k] = load_near16(Xq, first + static_cast<int64_t>(h0 + kb + k) * image_row, x_bytes);
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                if (kb + k >= KH) break;
                const int h = h0 + kb + k;
                const bool inside = static_cast<unsigned>(h) < static_cast<unsigned>(ct.H);
                a[k] = keep(a[k], Xq, first + static_cast<int64_t>(h) * image_row, x_bytes, inside ? lo : 16, hi, mask);
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const v4i w = *reinterpret_cast<const v4i*>(lds + (((kb + k) * FN + j) * 64 + lane) * 16);
                    acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[k], w, acc[j], 0, 0, 0);
                }
            }
        }
        // accumulator register r of lane l is pixel 8 * (r / 4) + 4 * (l / 32) + r % 4 of the tile, channel l % 32
        float* out = Y + static_cast<int64_t>(m0 + 4 * half) * Cout + col;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int dr = 8 * (r >> 2) + (r & 3);
            if (m0 + 4 * half + dr >= M) continue;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (32 * j + col >= Cout) continue;
                const float v = plain ? static_cast<float>(acc[j][r]) * unit : unmap_value(acc[j][r], E);
                __builtin_nontemporal_store(v, out + static_cast<int64_t>(dr) * Cout + 32 * j);
            }
        }
    }
}

int conv_thin_fwd_launch(const ConvTaps& ct, int KH, int64_t images, int64_t M, int64_t Cout, const int8_t* Xq, const int8_t* Wq,
                         float* Y, const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, hipStream_t s) {
    const int fn = static_cast<int>((Cout + 31) / 32);
    // a filter row is one 32-byte step, all output channels of a pixel belong to one wave, the weights fit the LDS
    if (ct.C > 4 || ct.KW * ct.C > 32 || fn > 4 || KH * fn > 64) return kNotApplicable;
    if (static_cast<int64_t>(ct.W) * ct.C >= (int64_t{1} << 28)) return kNotApplicable;          // 32-bit offsets in an image row
    const int64_t x_bytes = images * ct.H * ct.W * ct.C;
    if (x_bytes < 16 || Cout * KH * ct.KW * ct.C < 16) return kNotApplicable;
    const uint32_t tiles = static_cast<uint32_t>((M + 31) / 32);
    // as many workgroups as are resident (four per CU with up to 64 output channels, else two), which walk the tiles: the weights
    // are laid out once per workgroup (32 x 224 x 224 x 3 -> 64: 3136 workgroups 38.0 us, 2048 32.5, 1568 34.3, 1024 29.3, 784 33.2)
    const dim3 grid(std::min<uint32_t>((tiles + 3) / 4, fn <= 2 ? 1024 : 512)), block(256);
    const size_t lds = static_cast<size_t>(KH) * fn * 1024;
#define FXP_THIN(FN)                                                                                                        \
    hipLaunchKernelGGL((k_conv_thin_fwd<FN>), grid, block, lds, s, Xq, Wq, Y, ct, KH, static_cast<uint32_t>(M),               \
                       static_cast<int>(Cout), x_bytes, eA, bitsA, eB, bitsB, tiles)
    if (fn == 1) FXP_THIN(1);
    else if (fn == 2) FXP_THIN(2);
    else if (fn == 3) FXP_THIN(3);
    else FXP_THIN(4);
#undef FXP_THIN
    return launch_status();
}

constexpr int kWgradThreads = 512, kWgradWaves = kWgradThreads / 64;

// how a weight gradient is cut up
struct WgradGeo {
    ConvTaps ct;
    int KH, Cout, K;
    int all_rows;         // output rows of the batch
    int wg_rows;          // output rows of a workgroup, a run over the batch
    int rows;             // those of them, at most, whose image rows are in LDS together (never of two images)
    int lds_rows;         // image rows of such a unit
    int shift;            // columns the planes start left of the image (a multiple of the stride, padding or more)
    int planes;           // stride * C
    int q;                // dwords of a plane row (odd: the planes of one pixel start in different banks)
    int chunks;           // 16-pixel pieces per output row
};

// parts[slice][co][k] = sum over the slice's output pixels of dYqT[co][m] * patch[m][k].  A lane's A operand is 16
// neighbouring pixels of one output channel of dYqT, its B operand the same pixels of one tap and channel; pixels beyond
// the end of an output row are zero in A.  The eight waves take the pairs of pieces of a unit in turn, each with all
// FM * FK fragments (blockIdx.y: the next FK * 32 columns k), and add up through LDS at the end.  One workgroup per CU:
// with two of half the waves there are twice the slices to write and to sum (30 and 13 us against 22 and 9; 2205, 20
// and 123 through stored transposed patches).
template <int FM, int FK>
__global__ __launch_bounds__(kWgradThreads, 2) void k_conv_thin_wgrad(const int8_t* __restrict__ Xq, const int8_t* __restrict__ dYqT,
                                                            int32_t* __restrict__ parts, int64_t part_stride, int64_t M,
                                                            WgradGeo g) {
    extern __shared__ __attribute__((aligned(16))) uint32_t planes[];
    const ConvTaps& ct = g.ct;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
    const int row_dw = g.planes * g.q;                             // dwords of one image row
    const int image_row = ct.W * ct.C;
    const int k_first = static_cast<int>(blockIdx.y) * FK * 32;
    int k_at[FK], k_align[FK];
#pragma unroll
    for (int j = 0; j < FK; ++j) {
        const int k = min(k_first + 32 * j + col, g.K - 1);        // columns beyond K are not stored
        const int tap = k / ct.C, c = k - tap * ct.C, kh = tap / ct.KW, kw = tap - kh * ct.KW;
        const int x = kw - ct.padw + g.shift, i = x / ct.stride, phase = x - i * ct.stride;
        k_at[j] = kh * row_dw + (phase * ct.C + c) * g.q + (i >> 2);
        k_align[j] = i & 3;
    }
    const int64_t a_bytes = static_cast<int64_t>(g.Cout) * M;
    int64_t a_row[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) a_row[i] = static_cast<int64_t>(min(32 * i + col, g.Cout - 1)) * M;
    v16i acc[FM][FK];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FK; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    int row_first = static_cast<int>(blockIdx.x) * g.wg_rows;
    const int row_end = min(row_first + g.wg_rows, g.all_rows);
    while (row_first < row_end) {
        const int n = row_first / ct.Ho, ho0 = row_first - n * ct.Ho;
        const int rows_here = min(min(g.rows, ct.Ho - ho0), row_end - row_first);
        const int total = rows_here * g.chunks;                    // 16-pixel pieces of the unit
        const int64_t m_unit = static_cast<int64_t>(row_first) * ct.Wo;
        row_first += rows_here;
        auto piece_of = [&](int step, int& r, int& j) {            // piece of this half-wave in a step; r < 0: none
            const int p = 2 * (kWgradWaves * step + wave) + half;
            r = p / g.chunks;
            j = p - r * g.chunks;
            if (p >= total) { r = -1; j = 0; }
        };
        auto m_of = [&](int r, int j) { return m_unit + static_cast<int64_t>(max(r, 0)) * ct.Wo + 16 * j; };
        auto load_a = [&](int r, int j, v4i (&a)[FM]) {
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = load_near16(dYqT, a_row[i] + m_of(r, j), a_bytes);
        };
        auto keep_a = [&](int r, int j, v4i (&a)[FM]) {
            const int n_bytes = r < 0 ? 0 : min(16, ct.Wo - 16 * j);
            uint32_t mask[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) mask[d] = byte_mask(0, n_bytes - 4 * d);
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = keep(a[i], dYqT, a_row[i] + m_of(r, j), a_bytes, 0, n_bytes, mask);
        };
        const int steps = (total + 2 * kWgradWaves - 1) / (2 * kWgradWaves);
        int r, j;
        v4i a[FM], a_next[FM];
        piece_of(0, r, j);
        load_a(r, j, a);
        // image rows -> planes: dword q of plane (phase, c) holds columns w = (4 q + e) * stride + phase - shift
        __syncthreads();                                           // the last unit's planes are read no more
        const int h_first = ho0 * ct.stride - ct.pad;
        for (int item = lane; item < row_dw; item += 64) {
            const int p = item / g.q, q = item - p * g.q, phase = p / ct.C, c = p - phase * ct.C;
            const int8_t* at[4];                                   // of image row 0; columns outside are masked
            uint32_t mask = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int w = (4 * q + e) * ct.stride + phase - g.shift;
                if (static_cast<unsigned>(w) < static_cast<unsigned>(ct.W)) mask |= 0xffu << (8 * e);
                at[e] = Xq + (static_cast<int64_t>(n) * ct.H * ct.W + min(max(w, 0), ct.W - 1)) * ct.C + c;
            }
#pragma unroll 4
            for (int lr = wave; lr < g.lds_rows; lr += kWgradWaves) {
                const int h = h_first + lr;
                const int64_t row = static_cast<int64_t>(min(max(h, 0), ct.H - 1)) * image_row;
                uint32_t v = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) v |= static_cast<uint32_t>(static_cast<uint8_t>(at[e][row])) << (8 * e);
                planes[lr * row_dw + item] = static_cast<unsigned>(h) < static_cast<unsigned>(ct.H) ? v & mask : 0u;
            }
        }
        __syncthreads();
        for (int step = 0; step < steps; ++step) {
            const uint32_t* at = planes + max(r, 0) * ct.stride * row_dw + 4 * j;
            keep_a(r, j, a);
            piece_of(step + 1, r, j);                              // none behind the last step: a load that is not used
            load_a(r, j, a_next);
#pragma unroll
            for (int f = 0; f < FK; ++f) {
                uint32_t d[5];
#pragma unroll
                for (int e = 0; e < 5; ++e) d[e] = at[k_at[f] + e];
                v4i b;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    b[e] = static_cast<int>(__builtin_amdgcn_alignbyte(d[e + 1], d[e], static_cast<uint32_t>(k_align[f])));
#pragma unroll
                for (int i = 0; i < FM; ++i) acc[i][f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b, acc[i][f], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = a_next[i];
        }
    }
    // the waves' sums meet in LDS, [co][k] with FK * 32 columns
    __syncthreads();
    int32_t* sum = reinterpret_cast<int32_t*>(planes);
    for (int i = threadIdx.x; i < FM * 32 * FK * 32; i += kWgradThreads) sum[i] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FK; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                atomicAdd(sum + (32 * i + 8 * (r >> 2) + 4 * half + (r & 3)) * (FK * 32) + 32 * j + col, acc[i][j][r]);
    __syncthreads();
    int32_t* dst = parts + static_cast<int64_t>(blockIdx.x) * part_stride + k_first;
    const int cols_here = min(FK * 32, g.K - k_first);
    for (int co = wave; co < g.Cout; co += kWgradWaves)
        for (int k = lane; k < cols_here; k += 64) dst[static_cast<int64_t>(co) * g.K + k] = sum[co * (FK * 32) + k];
}

struct WgradPlan {
    WgradGeo g;
    int fm, fk, k_groups;      // fragments of output channels and of k per wave, groups of k fragments
    int slices;
    int64_t slice_stride;
    size_t lds;
};

static bool plan_thin_wgrad(const ConvTaps& ct, int KH, int64_t images, int64_t Cout, size_t part_bytes, WgradPlan* p) {
    if (ct.C > 4 || ct.KW * ct.C > 32 || Cout > 128 || ct.stride > 4) return false;
    WgradGeo& g = p->g;
    g.ct = ct;
    g.KH = KH;
    g.Cout = static_cast<int>(Cout);
    g.K = KH * ct.KW * ct.C;
    g.chunks = (ct.Wo + 15) / 16;
    g.shift = (ct.padw + ct.stride - 1) / ct.stride * ct.stride;
    g.planes = ct.stride * ct.C;
    const int i_max = (ct.KW - 1 - ct.padw + g.shift) / ct.stride;
    const int64_t q = (i_max / 4 + 4 * (static_cast<int64_t>(g.chunks) - 1) + 5) | 1;
    const int k_frags = (g.K + 31) / 32;
    p->fm = static_cast<int>((Cout + 31) / 32);
    // fragments of k per wave: all of them where 160 accumulator registers hold them
    const int fk_max = p->fm <= 2 ? 5 : (p->fm == 3 ? 3 : 2);
    p->fk = k_frags == 1 ? 1 : (k_frags == 2 || fk_max == 2 ? 2 : fk_max);
    p->k_groups = (k_frags + p->fk - 1) / p->fk;
    // One workgroup per CU with an equal run of output rows.  Image rows in LDS at a time: 48 KiB at most, for a run of up
    // to 16 output rows (rows of the filter that reach into the neighbouring unit are fetched by both).
    auto image_bytes = [&](int64_t rows) { return ((rows - 1) * ct.stride + KH) * g.planes * q * 4; };
    p->slice_stride = (Cout * g.K + 3) / 4 * 4;
    const int64_t all_rows = images * ct.Ho;
    const int64_t fit = static_cast<int64_t>(part_bytes / (static_cast<size_t>(p->slice_stride) * sizeof(int32_t)));
    const int64_t want = std::min<int64_t>({all_rows, int64_t{std::max(1, 256 / p->k_groups)}, fit});
    if (want < 1 || all_rows >= (int64_t{1} << 30)) return false;
    const int64_t wg_rows = (all_rows + want - 1) / want;
    int64_t rows = std::min<int64_t>({wg_rows, 16, ct.Ho});
    while (rows > 1 && image_bytes(rows) > 49152) --rows;
    // ... and every slice exact in int32
    if (image_bytes(rows) > 49152 || wg_rows * ct.Wo > kMaxSlice || images * ct.H * ct.W * ct.C < 16 || Cout * all_rows * ct.Wo < 16)
        return false;
    // A unit costs 1.1 us for each 32 output channels, however few its pixels; a stored patch costs by its bytes, taps next to
    // each other in a row more than one column of them, and little where a pixel's channels are one dword.  Many units of few
    // pixels are stored patches' (layer steps, image here / stored in us: 20000 x 2 x 2 x 1 -> 128 2x2 420 / 52, 10000 x 4 x 4 x 1
    // -> 16 1x1 92 / 66, 3000 x 7 x 7 x 3 -> 128 1x1 143 / 91, 64 x 4096 x 1 x 4 -> 64 3x1 270 / 79, 20000 x 4 x 4 x 4 -> 64 3x3
    // 219 / 108; on the other side 3000 x 7 x 7 x 1 -> 128 3x3 121 / 131, 64 x 4096 x 1 x 2 -> 16 5x1 171 / 206, 64 x 256 x 8 x 1
    // -> 16 1x1 43 / 58, 512 x 14 x 14 x 4 -> 64 3x3 52 / 59, 64 x 128 x 32 x 4 -> 64 3x1 equal).  One or two units save a launch.
    const int64_t pixels = rows * ct.Wo, patch = pixels * g.K * ct.KW;
    if (wg_rows > 2 * rows && (ct.C == 4 ? patch < 2048 * p->fm : pixels < 128 && patch < 156 * p->fm)) return false;
    g.all_rows = static_cast<int>(all_rows);
    g.wg_rows = static_cast<int>(wg_rows);
    g.rows = static_cast<int>(rows);
    g.q = static_cast<int>(q);
    g.lds_rows = static_cast<int>((rows - 1) * ct.stride + KH);
    p->slices = static_cast<int>((all_rows + wg_rows - 1) / wg_rows);
    p->lds = std::max<size_t>(static_cast<size_t>(image_bytes(rows)), static_cast<size_t>(p->fm) * p->fk * 4096);
    return true;
}

bool conv_thin_wgrad_fits(const ConvTaps& ct, int KH, int64_t images, int64_t Cout, size_t part_bytes) {
    WgradPlan p;
    return plan_thin_wgrad(ct, KH, images, Cout, part_bytes, &p);
}

// Leaves the slices in `parts` (16-byte aligned, part_bytes available) and describes in *sum the slices, to be completed
// by the caller with the output and the scales.
int conv_thin_wgrad_launch(const ConvTaps& ct, int KH, int64_t images, int64_t M, int64_t Cout, const int8_t* Xq, const int8_t* dYqT,
                           void* parts, size_t part_bytes, ReduceRider* sum, hipStream_t s) {
    WgradPlan p;
    if (!plan_thin_wgrad(ct, KH, images, Cout, part_bytes, &p)) return kNotApplicable;
    const dim3 grid(static_cast<unsigned>(p.slices), static_cast<unsigned>(p.k_groups)), block(kWgradThreads);
#define FXP_THIN(FM, FK)                                                                                                     \
    hipLaunchKernelGGL((k_conv_thin_wgrad<FM, FK>), grid, block, p.lds, s, Xq, dYqT, static_cast<int32_t*>(parts), p.slice_stride, \
                       M, p.g)
#define FXP_THIN_FK(FM, MAX)                 \
    do {                                     \
        if (p.fk == 1) FXP_THIN(FM, 1);      \
        else if (p.fk == 2) FXP_THIN(FM, 2); \
        else FXP_THIN(FM, MAX);              \
    } while (0)
    if (p.fm == 1) FXP_THIN_FK(1, 5);
    else if (p.fm == 2) FXP_THIN_FK(2, 5);
    else if (p.fm == 3) FXP_THIN_FK(3, 3);
    else FXP_THIN_FK(4, 2);
#undef FXP_THIN_FK
#undef FXP_THIN
    *sum = ReduceRider();
    sum->parts = static_cast<const int32_t*>(parts);
    sum->splits = p.slices;
    sum->stride = p.slice_stride;
    sum->M = static_cast<int>(Cout);
    sum->N = p.g.K;
    sum->ldc = p.g.K;
    sum->wide = M > kMaxContraction ? 1 : 0;
    return launch_status();
}

}  // namespace fxp
