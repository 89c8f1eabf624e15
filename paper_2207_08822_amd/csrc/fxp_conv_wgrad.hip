// Weight gradient of a convolution without stored patches (paper Sec. 3.4, App. A.2):
//   dW[co][(kh, kw, c)] = unmap( sum over output pixels m of dYq[m][co] * Xq[pixel of m under tap (kh, kw)][c] )
//
// Both operands lie with the channels contiguous and the contraction (the pixels) across, and a tap shifts the pixels by single
// rows, so they cannot be read contraction-contiguous from memory.  They are staged as they lie - one LDS row per pixel, 16-byte
// pieces along the channels, straight from the image or from a page of zeros - and transposed on the way to the matrix cores:
// ds_read_b64_tr_b8 hands lane j of 16 the bytes of column j of eight rows, so two of them make the 16 contraction bytes a lane of
// v_mfma_i32_32x32x32_i8 holds.  Channels on both sides in multiples of 16 (whole pieces).
//
// Before, the patches were transposed into memory (k_im2col_t_i8) and multiplied from there, contraction-contiguous.  32 x 28 x 28
// x 128, 3x3 (25088 pixels): 12.3 us to write 29 MB of them, with the block maxima of dY in the same launch, and 11.5 for the
// product; now 4.2 for the maxima and 12.4 for the product, step 63.0 -> 54.9 us; 64 x 56 x 56 x 64 140 -> 111, 256 x 28 x 28 x 128
// 331 -> 225, 8 x 224 x 224 x 16 235 -> 203.  Bound by the LDS and by what the barriers leave unoverlapped: a step of 128 pixels
// takes 0.75 us, of which 96 KiB read from LDS 0.32 and 32 KiB written 0.11, the matrix cores 0.21 (five stages for four:
// slower, so it is not the latency of the loads).
#include <algorithm>

#include "fxp_gemm_device.h"
#include "fxp_gemm_plan.h"
#include "fxp_internal.h"

namespace fxp {

typedef int v2i __attribute__((ext_vector_type(2)));

struct WgradArgs {
    const int8_t* G;          // [M][Cout]
    const int8_t* X;          // [N][H][W][C]
    void* out;                // [Cout][K], or slices of it
    int M, Cout, K;
    int per_slice;            // pixels of a slice, a multiple of the step
    int64_t split_stride;
    const int32_t* eA;
    const int32_t* eB;
    int bitsA, bitsB;
    int tiles_m, tiles_n, slices;
    int step_n, step_h, step_w;      // how far kStep pixels lead: images, rows, columns
};

constexpr int kStep = kWgradStep;    // pixels of a stage

// Half a wave of a transposing read meets eight rows of 32 bytes: pairs of 16-byte pieces are exchanged so that these fall into
// all 64 banks once (single pieces exchanged as in the other product kernels: two-way conflicts, half of the LDS's time).
template <int ROW_BYTES>
__device__ inline int pair_swizzle(int row) {
    return ROW_BYTES == 128 ? 2 * ((row >> 1) & 3) : 2 * ((row >> 2) & 1);
}

// BM output channels x BN weights of a channel, WM x WN of them a wave
template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void k_conv_wgrad(WgradArgs g, ConvTaps ct) {
    constexpr int NW = (BM / WM) * (BN / WN);
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int A_BYTES = kStep * BM, STAGE_BYTES = kStep * (BM + BN);
    constexpr int CPA = BM / 16, CPB = BN / 16;                  // 16-byte pieces of an LDS row
    constexpr int A_LOADS = A_BYTES / 1024 / NW, B_LOADS = kStep * BN / 1024 / NW, LOADS = A_LOADS + B_LOADS;
    static_assert(A_BYTES % (1024 * NW) == 0 && kStep * BN % (1024 * NW) == 0, "regions divide over the waves");
    static_assert((STAGES - 1) * LOADS < 64, "vmcnt is a 6-bit counter");
    __shared__ __attribute__((aligned(1024))) int8_t lds[STAGES * STAGE_BYTES];

    // a run of (slice, tile) pairs per XCD, slice-major: the tiles of a slice read the same pixels
    const int tiles = g.tiles_m * g.tiles_n, total = tiles * g.slices, v = static_cast<int>(blockIdx.x);
    const int q = total / kNumXcd, r = total % kNumXcd, xcd = v % kNumXcd, local = v / kNumXcd;
    const int p = xcd < r ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
    const int slice = p / tiles, t = p - slice * tiles, tn = t / g.tiles_m, tm = t - tn * g.tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;
    const int first = slice * g.per_slice, end = min(g.M, first + g.per_slice);
    const int steps = (end - first + kStep - 1) / kStep;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = wave / (BN / WN) * WM, wn0 = wave % (BN / WN) * WN;
    const int8_t* const zeros = reinterpret_cast<const int8_t*>(g_zero_page);

    // Where this lane's pieces come from (beyond the last channel or weight: the last piece, for products that are not stored).
    // The gradient: its pixel row of the stage, its channels ...
    const int8_t* ga[A_LOADS];
    int a_row[A_LOADS];
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) {
        const int row = (wave + j * NW) * (64 / CPA) + lane / CPA;
        const int col = min(m0 + 16 * ((lane % CPA) ^ pair_swizzle<BM>(row)), g.Cout - 16);
        a_row[j] = row;
        ga[j] = g.G + static_cast<int64_t>(first + row) * g.Cout + col;
    }
    // ... and the image: the input pixel (h, w) of its output pixel under its tap, and that pixel's offset from the first image of
    // the slice; what a step adds to them, by itself and where the output pixel passes the end of a line or of an image
    const int lines0 = first / ct.Wo, image0 = lines0 / ct.Ho;                       // workgroup-uniform
    const int8_t* const x0 = g.X + static_cast<int64_t>(image0) * ct.H * ct.W * ct.C;
    int b_row[B_LOADS], b_h[B_LOADS], b_w[B_LOADS], b_off[B_LOADS], b_hend[B_LOADS], b_wend[B_LOADS];
    const int line_w = ct.Wo * ct.stride, line_h = ct.Ho * ct.stride, move_w = g.step_w * ct.stride, move_h = g.step_h * ct.stride;
    const int row_bytes = ct.W * ct.C;
    const int off_step = (g.step_n * ct.H + move_h) * row_bytes + move_w * ct.C;
    const int off_line = ct.stride * row_bytes - line_w * ct.C, off_image = (ct.H - line_h) * row_bytes;
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
        const int row = (wave + j * NW) * (64 / CPB) + lane / CPB;
        const int n = min(n0 + 16 * ((lane % CPB) ^ pair_swizzle<BN>(row)), g.K - 16);
        const int tap = n / ct.C, kh = tap / ct.KW, dh = kh - ct.pad, dw = tap - kh * ct.KW - ct.padw;
        const uint32_t m = static_cast<uint32_t>(first + row), line = m / static_cast<uint32_t>(ct.Wo);
        const uint32_t image = line / static_cast<uint32_t>(ct.Ho);
        b_row[j] = row;
        b_w[j] = static_cast<int>(m - line * ct.Wo) * ct.stride + dw;
        b_h[j] = static_cast<int>(line - image * ct.Ho) * ct.stride + dh;
        b_off[j] = ((static_cast<int>(image) - image0) * ct.H + b_h[j]) * row_bytes + b_w[j] * ct.C + n - tap * ct.C;
        b_wend[j] = line_w + dw;
        b_hend[j] = line_h + dh;
    }
    // the next stage to be loaded, in order; moves the rows on by kStep pixels
    const int64_t a_step = static_cast<int64_t>(kStep) * g.Cout;
    int loaded = 0;
    auto issue = [&](int stage) {
        int8_t* const st = lds + stage * STAGE_BYTES;
        const int left = end - first - loaded;                                       // workgroup-uniform
        loaded += kStep;
        const int8_t* src_a[A_LOADS];
        const int8_t* src_b[B_LOADS];
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j) {
            src_a[j] = ga[j];
            ga[j] += a_step;
        }
#pragma unroll
        for (int j = 0; j < B_LOADS; ++j) {
            const bool inside = static_cast<unsigned>(b_h[j]) < static_cast<unsigned>(ct.H) &&
                                static_cast<unsigned>(b_w[j]) < static_cast<unsigned>(ct.W);
            src_b[j] = inside ? x0 + b_off[j] : zeros;
            b_w[j] += move_w;
            const bool line = b_w[j] >= b_wend[j];
            b_w[j] -= line ? line_w : 0;
            b_h[j] += move_h + (line ? ct.stride : 0);
            const bool image = b_h[j] >= b_hend[j];
            b_h[j] -= image ? line_h : 0;
            b_off[j] += off_step + (line ? off_line : 0) + (image ? off_image : 0);
        }
        if (left < kStep) {                                                          // the last stage of the last slice
#pragma unroll
            for (int j = 0; j < A_LOADS; ++j)
                if (a_row[j] >= left) src_a[j] = zeros;
#pragma unroll
            for (int j = 0; j < B_LOADS; ++j)
                if (b_row[j] >= left) src_b[j] = zeros;
        }
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src_a[j],
                                             (__attribute__((address_space(3))) void*)(st + (wave + j * NW) * 1024), 16, 0, 0);
#pragma unroll
        for (int j = 0; j < B_LOADS; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src_b[j],
                                             (__attribute__((address_space(3))) void*)(st + A_BYTES + (wave + j * NW) * 1024), 16, 0, 0);
    };

    // Fragments of 32 pixels: lane 16 g + i reads 8 bytes of pixel row 16 (g / 2) + 8 t + i / 2, 16-byte piece g % 2 of the
    // fragment's 32 channels, half i % 2, and receives column i of its group's piece.
    const int i16 = lane & 15, group = lane >> 4;
    int a_at[FM][2], b_at[FN][2];
#pragma unroll
    for (int t8 = 0; t8 < 2; ++t8) {
        const int row = 16 * (group >> 1) + 8 * t8 + (i16 >> 1);              // (the swizzle repeats every 16 rows or fewer)
#pragma unroll
        for (int i = 0; i < FM; ++i)
            a_at[i][t8] = row * BM + 16 * (((wm0 + 32 * i) / 16 + (group & 1)) ^ pair_swizzle<BM>(row)) + 8 * (i16 & 1);
#pragma unroll
        for (int j = 0; j < FN; ++j)
            b_at[j][t8] = A_BYTES + row * BN + 16 * (((wn0 + 32 * j) / 16 + (group & 1)) ^ pair_swizzle<BN>(row)) + 8 * (i16 & 1);
    }
    auto transposed = [&](const int8_t* at) {
        return __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i*)at);
    };
    v16i acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;
    constexpr int KS = kStep / 32;
    v4i fa[2][FM], fb[2][FN];
    auto read_frags = [&](int buf, int stage, int ks) {
        const int8_t* st = lds + stage * STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const v2i lo = transposed(st + a_at[i][0] + ks * 32 * BM), hi = transposed(st + a_at[i][1] + ks * 32 * BM);
            fa[buf][i] = v4i{lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const v2i lo = transposed(st + b_at[j][0] + ks * 32 * BN), hi = transposed(st + b_at[j][1] + ks * 32 * BN);
            fb[buf][j] = v4i{lo[0], lo[1], hi[0], hi[1]};
        }
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
    };
    auto barrier = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // the schedule of k_gemm_nt_dma: the barrier that publishes the next stage stands before the last 32 pixels of this one
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < steps) issue(s);
    if (steps >= STAGES) wait_loads_and_lds<(STAGES - 1) * LOADS>();
    else wait_loads_and_lds<0>();
    barrier();
    read_frags(0, 0, 0);
    auto stage_body = [&](int it, auto wait_next, auto refill) {
        const int stage = it % STAGES;
#pragma unroll
        for (int ks = 0; ks + 1 < KS; ++ks) {
            read_frags((ks & 1) ^ 1, stage, ks + 1);
            multiply(ks & 1);
        }
        wait_next();
        barrier();
        read_frags(0, (it + 1) % STAGES, 0);
        refill(stage);
        multiply(1);
    };
    auto steady_wait = [] { wait_loads_and_lds<(STAGES - 2) * LOADS>(); };
    auto full_wait = [] { wait_loads_and_lds<0>(); };
    auto no_refill = [](int) {};
    int it = 0;
    for (; it + STAGES < steps; ++it) stage_body(it, steady_wait, issue);
    for (; it + STAGES - 1 < steps; ++it) stage_body(it, steady_wait, no_refill);
    for (; it + 1 < steps; ++it) stage_body(it, full_wait, no_refill);
    const int stage = (steps - 1) % STAGES;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) read_frags((ks & 1) ^ 1, stage, ks + 1);
        multiply(ks & 1);
    }
    int E = 0;
    if (MODE == kStoreF32) E = lsb_exponent(g.eA[0], g.bitsA) + lsb_exponent(g.eB[0], g.bitsB);
    store_fragments<FM, FN, MODE, false>(acc, static_cast<int32_t*>(g.out) + static_cast<int64_t>(slice) * g.split_stride, g.K, g.Cout,
                                         g.K, m0 + wm0, n0 + wn0, lane >> 5, lane & 31, E);
}

// ws: WgradCut::ws_bytes for the slices, 16-byte aligned.
int conv_wgrad_launch(const ConvTaps& ct, int KH, int64_t M, int64_t Cout, const int8_t* Xq, const int8_t* dYq, float* dW,
                      const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, void* ws, hipStream_t s, ReduceRider* defer) {
    const int64_t K = static_cast<int64_t>(KH) * ct.KW * ct.C;
    const WgradCut p = plan_conv_wgrad(M, Cout, K);
    const int64_t stride = (Cout * K + 3) / 4 * 4;
    WgradArgs g;
    g.G = dYq; g.X = Xq;
    g.M = static_cast<int>(M); g.Cout = static_cast<int>(Cout); g.K = static_cast<int>(K);
    g.per_slice = static_cast<int>(p.per_slice);
    g.slices = p.slices;
    g.tiles_m = p.tiles_m; g.tiles_n = p.tiles_n;
    g.split_stride = stride;
    g.eA = eA; g.bitsA = bitsA; g.eB = eB; g.bitsB = bitsB;
    const int area = ct.Ho * ct.Wo, rest = kStep % area;
    g.step_n = kStep / area;
    g.step_h = rest / ct.Wo;
    g.step_w = rest % ct.Wo;
    g.out = p.slices > 1 ? ws : dW;
    const dim3 grid(static_cast<unsigned>(p.tiles_m) * p.tiles_n * p.slices), block(p.pairs ? 256 : 512);
#define FXP_WGRAD_LAUNCH(BM, WM, WN, STAGES)                                                                                         \
    do {                                                                                                                             \
        if (p.slices > 1) hipLaunchKernelGGL((k_conv_wgrad<BM, 128, WM, WN, STAGES, kStoreI32>), grid, block, 0, s, g, ct);           \
        else hipLaunchKernelGGL((k_conv_wgrad<BM, 128, WM, WN, STAGES, kStoreF32>), grid, block, 0, s, g, ct);                        \
    } while (0)
    if (p.bm == 64) FXP_WGRAD_LAUNCH(64, 32, 32, 4);
    else if (p.pairs) FXP_WGRAD_LAUNCH(128, 64, 64, 2);
    else FXP_WGRAD_LAUNCH(128, 64, 32, 4);
#undef FXP_WGRAD_LAUNCH
    const int rc = launch_status();
    if (rc || p.slices == 1) return rc;
    ReduceRider r;
    r.parts = static_cast<const int32_t*>(ws);
    r.splits = p.slices;
    r.stride = stride;
    r.M = g.Cout; r.N = g.K;
    r.C = dW; r.ldc = K;
    r.fp32_out = 1;
    r.eA = eA; r.bitsA = bitsA; r.eB = eB; r.bitsB = bitsB;
    r.wide = M > kMaxContraction ? 1 : 0;
    // (a rider takes a lane a piece: more slices than that are summed by several, in a launch of their own)
    if (defer == nullptr || p.slices > 64) return splitk_reduce_launch(r, s);
    r.blocks = static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(2048, (Cout * K / 4 + 255) / 256)));
    *defer = r;
    return FXP_OK;
}

// Channels in whole 16-byte pieces, 32-bit pixel numbers and offsets in a slice's images, room for the slices, no 1x1 layer of few
// pixels (one_tap_patches); up to 512 tiles, which is what is resident at once of the two-per-CU kernel: beyond, the larger tiles of the
// product of stored patches are ahead where there are pixels enough (stored / from the image in us: 576 tiles, 16 x 14 x 14 x 1024
// 3x3 127 / 146, 64 x 7 x 7 127 / 146, but 16 x 7 x 7 86 / 81; 567, 16 x 14 x 14 x 896 -> 1152 122 / 143; 441, 896 -> 896 119 / 100).
// The kernels with one workgroup a CU gain up to there as well, in two rounds (432 tiles, 32 x 14 x 14 x 6144 -> 64 549 / 420; 270,
// 64 x 14 x 14 x 640 -> 768 239 / 205).
bool conv_wgrad_fits(const ConvTaps& ct, int KH, int64_t M, int64_t Cout, size_t ws_bytes) {
    if (ct.C % 16 != 0 || Cout % 16 != 0 || M >= (int64_t{1} << 30)) return false;
    if (KH == 1 && ct.KW == 1 && one_tap_patches(M, Cout, ct.C)) return false;
    const WgradCut p = plan_conv_wgrad(M, Cout, static_cast<int64_t>(KH) * ct.KW * ct.C);
    return static_cast<int64_t>(p.tiles_m) * p.tiles_n <= 512 && p.ws_bytes <= ws_bytes &&
           (p.per_slice / (static_cast<int64_t>(ct.Ho) * ct.Wo) + 4) * ct.H * ct.W * ct.C < (int64_t{1} << 31);
}

}  // namespace fxp
