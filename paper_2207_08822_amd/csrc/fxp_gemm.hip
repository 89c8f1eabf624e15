// Integer GEMM on the matrix cores (paper Sec. 3.3, Fig. 2: int8 x int8 products,
// int32 accumulation) with the non-linear inverse mapping of Sec. 3.2 fused into the
// epilogue.
//
// One kernel form: C[M,N] = A[M,K] * B[N,K]^T with BOTH operands contiguous along the
// contraction (the mapping kernel emits every tensor in both orientations, so the three
// GEMMs of a layer step all take this form).  v_mfma_i32_32x32x32_i8: a lane holds 16
// consecutive contraction bytes of one row (A) or one column (B); integer addition is
// order-free, so only "same bytes on both sides" matters for the contraction index.
//
//   * three kernels share the tile scheme and the epilogue: k_gemm_nt stages tiles through registers (two LDS
//     buffers, any alignment and leading dimension: the fallback), k_gemm_nt_dma loads global -> LDS directly in a
//     multi-stage pipeline (the workhorse for every tile shape but the largest), k_gemm_nt_ring keeps a five-slot
//     ring of 256 x 256 x 128 tiles for the MFMA-bound shapes;
//   * LDS rows are BK bytes; 16-byte pieces are XOR-swizzled by the row so that the
//     64-lane ds_read_b128 of a fragment (32 rows x 2 pieces) spreads over all banks;
//   * accumulator lanes run along N: each store instruction writes 128-byte runs;
//   * workgroups are renumbered so that each XCD (own L2) works on a compact patch of
//     tiles instead of every 8th tile;
//   * long-contraction / small-output shapes split K across grid.y: every slice stores its int32 tile into a
//     workspace slice and a reduction (its own launch, or riding in the next product's) sums them and applies the
//     inverse mapping; without workspace the slices add into C with int32 atomics (exact either way: integer
//     addition is associative).
// Roofline: MFMA-bound when 2MNK / (MK + NK + 4MN bytes) is above ~630 ops/B, else HBM.
#include <algorithm>
#include <type_traits>

#include "fxp_gemm_device.h"
#include "fxp_gemm_plan.h"
#include "fxp_internal.h"

namespace fxp {

// batched product: `count` matrices, element strides between consecutive ones (grid.z)
struct Batch {
    unsigned count = 1;
    int64_t a = 0, b = 0, c = 0;
};

// Workgroup b runs on XCD b % 8.  Give XCD x the contiguous range of tile numbers
// [start(x), start(x+1)), then walk tiles in column-major groups of `group_m` tile rows
// so that concurrently resident tiles share A and B panels in that XCD's L2.
__device__ inline void tile_of_block(int b, int tiles_m, int tiles_n, int group_m, int* tm, int* tn) {
    const int total = tiles_m * tiles_n;
    const int q = total / kNumXcd, r = total % kNumXcd;
    const int xcd = b % kNumXcd, local = b / kNumXcd;
    const int t = (xcd < r) ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
    const int per_group = group_m * tiles_n;
    const int g = t / per_group, in_g = t % per_group;
    const int rows_here = min(group_m, tiles_m - g * group_m);
    *tm = g * group_m + in_g % rows_here;
    *tn = in_g / rows_here;
}

// Sum of the split-K slices of a product (exact in any order) -> int32 or inverse-mapped fp32, by workgroup
// `b` of `nb`.  The slices are dense M x N matrices `stride` elements apart.  A dense, 16-byte aligned output is
// walked as one flat run of 16-byte pieces, anything else row by row.  ALONE: a launch of its own, which may share a piece
// among lanes; a rider in a product's launch takes a lane a piece (with the shared pieces in every product kernel, and twice
// the riders, the input gradient of a 32 x 28 x 28 x 128 3x3 layer took 14.0 us for 11.3).  64-bit sums ride like any other:
// layer steps of 64 x 56 x 56 x 64 -> 64 3x3 145 us, with a launch of their own 151, one element a thread 176;
// 262144 x 128 x 512 521 / 528 / 525; 200000 x 256 x 64 230 / 241 / 264.
// NT: threads of the workgroup, 256 alone, those of the host product when riding (blockDim would be a vector load).
template <bool ALONE, unsigned NT>
__device__ inline void splitk_reduce_body(const ReduceRider& r, unsigned b, unsigned nb) {
    constexpr unsigned nt = NT;
    float m = 0.0f;
    int E = 0;
    if (r.fp32_out) E = lsb_exponent(r.eA[0], r.bitsA) + (r.eB ? lsb_exponent(r.eB[0], r.bitsB) : 0);
    const int32_t* __restrict__ parts = r.parts;
    const int64_t stride = r.stride;
    const int splits = r.splits;
    auto one = [&](int acc, int32_t* dst) {
        if (r.fp32_out) {
            const float o = unmap_value(acc, E);
            *reinterpret_cast<float*>(dst) = o;
            m = fmaxf(m, fabsf(o));
        } else {
            *dst = acc;
        }
    };
    const int64_t total = static_cast<int64_t>(r.M) * r.N;
    const bool flat = r.ldc == r.N && (reinterpret_cast<uintptr_t>(r.C) & 15u) == 0;
    // 16-byte pieces of a flat output: `group` lanes of a wave share a piece, each sums every group-th slice, and the
    // lanes add up by exchange
    auto pieces = [&](auto wide_c) {
        constexpr bool WIDE = decltype(wide_c)::value != 0;
        using Sum = typename std::conditional<WIDE, int64_t, int>::type;
        const int lane = threadIdx.x & 63, per_wave = 64 / r.group, sub = lane / per_wave;
        const int64_t nvec = total >> 2, waves = static_cast<int64_t>(nb) * (nt >> 6);
        int64_t i = (static_cast<int64_t>(b) * (nt >> 6) + (threadIdx.x >> 6)) * per_wave + lane % per_wave;
        for (; i < nvec; i += waves * per_wave) {                  // the lanes of one piece leave together
            Sum s[4] = {0, 0, 0, 0};
#pragma unroll 8
            for (int sidx = sub; sidx < splits; sidx += r.group) {
                const int4 v = reinterpret_cast<const int4*>(parts + sidx * stride)[i];
                s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
            }
            for (int d = per_wave; d < 64; d *= 2)
#pragma unroll
                for (int k = 0; k < 4; ++k) s[k] += __shfl_xor(s[k], d);
            if (sub != 0) continue;
            if (r.fp32_out) {
                float o[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if constexpr (WIDE) o[k] = unmap_value64(s[k], E);
                    else o[k] = unmap_value(s[k], E);
                    m = fmaxf(m, fabsf(o[k]));
                }
                reinterpret_cast<float4*>(r.C)[i] = make_float4(o[0], o[1], o[2], o[3]);
            } else {
                reinterpret_cast<int4*>(r.C)[i] =
                    make_int4(static_cast<int>(s[0]), static_cast<int>(s[1]), static_cast<int>(s[2]), static_cast<int>(s[3]));
            }
        }
    };
    // the same with a lane a piece
    auto wide_pieces = [&]() {
        for (int64_t i = static_cast<int64_t>(b) * nt + threadIdx.x; i < total >> 2; i += static_cast<int64_t>(nb) * nt) {
            int64_t s[4] = {0, 0, 0, 0};
#pragma unroll 8
            for (int sidx = 0; sidx < splits; ++sidx) {
                const int4 v = reinterpret_cast<const int4*>(parts + sidx * stride)[i];
                s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
            }
            float o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                o[k] = unmap_value64(s[k], E);
                m = fmaxf(m, fabsf(o[k]));
            }
            reinterpret_cast<float4*>(r.C)[i] = make_float4(o[0], o[1], o[2], o[3]);
        }
    };
    if (r.wide) {
        // contraction beyond what one int32 sum holds: 64-bit sums of the slices
        int64_t i = static_cast<int64_t>(b) * nt + threadIdx.x;
        if (flat) {
            if constexpr (ALONE) pieces(IC<1>{});
            else wide_pieces();
            i += total & ~int64_t{3};                               // the tail, one element per thread
        }
        for (; i < total; i += static_cast<int64_t>(nb) * nt) {
            int64_t acc = 0;
            for (int sidx = 0; sidx < splits; ++sidx) acc += parts[sidx * stride + i];
            const float o = unmap_value64(acc, E);
            static_cast<float*>(r.C)[(i / r.N) * r.ldc + i % r.N] = o;
            m = fmaxf(m, fabsf(o));
        }
    } else if (flat) {
        const int64_t nvec = total >> 2;
        if (ALONE && r.group > 1) {
            pieces(IC<0>{});
        } else {
            for (int64_t i = static_cast<int64_t>(b) * nt + threadIdx.x; i < nvec; i += static_cast<int64_t>(nb) * nt) {
                int4 acc = make_int4(0, 0, 0, 0);
#pragma unroll 8
                for (int sidx = 0; sidx < splits; ++sidx) {
                    const int4 v = reinterpret_cast<const int4*>(parts + sidx * stride)[i];
                    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
                }
                if (r.fp32_out) {
                    float4 o;
                    o.x = unmap_value(acc.x, E); o.y = unmap_value(acc.y, E);
                    o.z = unmap_value(acc.z, E); o.w = unmap_value(acc.w, E);
                    reinterpret_cast<float4*>(r.C)[i] = o;
                    m = fmaxf(fmaxf(m, fmaxf(fabsf(o.x), fabsf(o.y))), fmaxf(fabsf(o.z), fabsf(o.w)));
                } else {
                    reinterpret_cast<int4*>(r.C)[i] = acc;
                }
            }
        }
        if (b == 0 && threadIdx.x < (total & 3)) {                 // the slices are 16-byte aligned, the tail is not a piece
            const int64_t i = (nvec << 2) + threadIdx.x;
            int acc = 0;
            for (int sidx = 0; sidx < splits; ++sidx) acc += parts[sidx * stride + i];
            one(acc, static_cast<int32_t*>(r.C) + i);
        }
    } else {
        for (int row = static_cast<int>(b); row < r.M; row += static_cast<int>(nb)) {
            const int32_t* prow = parts + static_cast<int64_t>(row) * r.N;
            int32_t* crow = static_cast<int32_t*>(r.C) + static_cast<int64_t>(row) * r.ldc;
            for (int i = threadIdx.x; i < r.N; i += static_cast<int>(nt)) {
                int acc = 0;
                for (int sidx = 0; sidx < splits; ++sidx) acc += prow[sidx * stride + i];
                one(acc, crow + i);
            }
        }
    }
    if (r.fp32_out && r.amax != nullptr) publish_absmax(m, r.amax);
}

// 16 bytes at any address (global memory takes 16-byte accesses at byte alignment)
struct __attribute__((packed, aligned(1))) Bytes16 {
    uint32_t x, y, z, w;
};
__device__ inline uint4 load16(const int8_t* p) {
    const Bytes16 b = *reinterpret_cast<const Bytes16*>(p);
    return make_uint4(b.x, b.y, b.z, b.w);
}

// v with its first n bytes (1 <= n <= 15) set to zero
__device__ inline uint4 clear_low_bytes(uint4 v, int n) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int c = min(max(n - 4 * d, 0), 4);                  // bytes of this dword that go
        w[d] = c == 4 ? 0u : w[d] >> (8 * c) << (8 * c);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// one product of a launch that may hold two
struct Product {
    const int8_t* A = nullptr;
    const int8_t* B = nullptr;
    void* C = nullptr;
    int64_t lda = 0, ldb = 0, ldc = 0;
    int M = 0, N = 0, K = 0;
    const int32_t* eA = nullptr;
    const int32_t* eB = nullptr;
    int bitsA = 8, bitsB = 8;
    uint32_t* amax = nullptr;
    int64_t batch_a = 0, batch_b = 0, batch_c = 0;
    int tiles_m = 0, tiles_n = 0;
    unsigned tiles = 0;      // 0: no product
};

// Products whose operands the direct-to-LDS kernels cannot take (rows that are not 16-byte aligned, or a contraction
// that is no multiple of 16): tiles are staged through registers, two steps ahead of the multiplication, into two LDS
// buffers.  A 16-byte piece is one load at whatever byte address its row starts (the ragged shapes pay in cache-line
// crossings, not in instructions: with one byte per load the products of a 1379 x 768 x 1000 layer took 198 and 100 us,
// now 13.1 and 8.6; the 96 products 197 x 64 x 197 of an attention block 22.2, now 6.5).  The last, partial piece of a
// row is read as the row's last 16 bytes on both operands - the contraction index may be permuted as long as both sides
// agree - and A's copies of bytes an earlier piece already brought are zeroed, so no load leaves the row.
// A contraction of one step (K <= BK) needs neither the second set of registers nor the second buffer: twice the workgroups
// per CU (the attention step of 4096 x (32 x 32 x 32): 157 us before there was a second set, 202 with both, 164 without).
// STEPS: kManySteps, kOneStep, or kOneStepBytes, a contraction shorter than 16 whose pieces are assembled byte by byte.
constexpr int kManySteps = 0, kOneStep = 1, kOneStepBytes = 2;
template <int BM, int BN, int BK, int WM, int WN, int STEPS, int MODE>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void k_gemm_nt(
    const int8_t* __restrict__ A, int64_t lda, const int8_t* __restrict__ B, int64_t ldb, void* __restrict__ Cv,
    int64_t ldc, int M, int N, int K, int k_per_split, const int32_t* __restrict__ eA, int bitsA,
    const int32_t* __restrict__ eB, int bitsB, int tiles_m, int tiles_n, int group_m, int64_t split_stride,
    int64_t batch_a, int64_t batch_b, int64_t batch_c, uint32_t* __restrict__ amax, ReduceRider rider, Product two) {
    int tile_block = static_cast<int>(blockIdx.x);
    if (rider.blocks != 0) {                                      // workgroup-uniform
        const unsigned first = rider.front ? 0u : rider.tiles;    // the riders are the first or the last workgroups
        if (blockIdx.x >= first && blockIdx.x < first + rider.blocks) {
            splitk_reduce_body<false, (BM / WM) * (BN / WN) * 64>(rider, blockIdx.x - first, rider.blocks);
            return;
        }
        if (rider.front) tile_block -= static_cast<int>(rider.blocks);
    }
    if (two.tiles != 0 && tile_block >= tiles_m * tiles_n) {      // workgroup-uniform: a tile of the second product
        tile_block -= tiles_m * tiles_n;
        A = two.A; B = two.B; Cv = two.C;
        lda = two.lda; ldb = two.ldb; ldc = two.ldc;
        M = two.M; N = two.N; K = two.K;
        k_per_split = two.K;
        eA = two.eA; eB = two.eB;
        bitsA = two.bitsA; bitsB = two.bitsB;
        amax = two.amax;
        batch_a = two.batch_a; batch_b = two.batch_b; batch_c = two.batch_c;
        tiles_m = two.tiles_m; tiles_n = two.tiles_n;
    }
    constexpr int NT = (BM / WM) * (BN / WN) * 64;
    constexpr int CPR = BK / 16;
    constexpr int NA = BM * CPR / NT, NB = BN * CPR / NT;   // 16-byte pieces per thread per step
    constexpr int FM = WM / 32, FN = WN / 32;               // 32x32 fragments per wave
    static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile does not divide over the threads");
    constexpr bool WIDE = STEPS != kOneStepBytes;
    constexpr int BUFS = STEPS == kManySteps ? 2 : 1;

    __shared__ __attribute__((aligned(16))) int8_t lds[BUFS][(BM + BN) * BK];

    int tm, tn;
    tile_of_block(tile_block, tiles_m, tiles_n, group_m, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int kb = blockIdx.y * k_per_split;
    // split-K into a workspace: slice y owns its own M x N int32 matrix (split_stride elements apart)
    Cv = static_cast<int32_t*>(Cv) + static_cast<int64_t>(blockIdx.y) * split_stride + static_cast<int64_t>(blockIdx.z) * batch_c;
    // batched product: matrix z of each operand lies batch_* elements further on
    A += static_cast<int64_t>(blockIdx.z) * batch_a;
    B += static_cast<int64_t>(blockIdx.z) * batch_b;
    const int ke = min(K, kb + k_per_split);
    const int nk = (ke - kb + BK - 1) / BK;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave / (BN / WN)) * WM, wn0 = (wave % (BN / WN)) * WN;

    // ---- global -> register staging ------------------------------------------------
    const int8_t* pa[NA];
    const int8_t* pb[NB];
    int lds_a[NA], lds_b[NB], kc_a[NA], kc_b[NB];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int id = tid + j * NT, row = id / CPR, c = id % CPR;
        pa[j] = A + static_cast<int64_t>(min(m0 + row, M - 1)) * lda;
        lds_a[j] = row * BK + ((c ^ swizzle_of_row<BK>(row)) * 16);
        kc_a[j] = c * 16;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int id = tid + j * NT, row = id / CPR, c = id % CPR;
        pb[j] = B + static_cast<int64_t>(min(n0 + row, N - 1)) * ldb;
        lds_b[j] = BM * BK + row * BK + ((c ^ swizzle_of_row<BK>(row)) * 16);
        kc_b[j] = c * 16;
    }
    uint4 ra[BUFS][NA], rb[BUFS][NB];

    // the piece of row p whose first contraction index is k, in a step that reaches the end of the slice
    auto tail_piece = [&](const int8_t* p, int k, bool clear) -> uint4 {
        if (WIDE) {
            if (k >= ke) return make_uint4(0, 0, 0, 0);
            const int from = min(k, ke - 16);
            const uint4 v = load16(p + from);
            return clear && from < k ? clear_low_bytes(v, k - from) : v;
        }
        uint32_t w[4] = {0, 0, 0, 0};
        for (int b = 0; b < 16; ++b)
            if (k + b < ke) w[b >> 2] |= static_cast<uint32_t>(static_cast<uint8_t>(p[k + b])) << (8 * (b & 3));
        return make_uint4(w[0], w[1], w[2], w[3]);
    };
    auto load_whole = [&](int it, uint4 (&va)[NA], uint4 (&vb)[NB]) {
        const int kk = kb + it * BK;
#pragma unroll
        for (int j = 0; j < NA; ++j) va[j] = load16(pa[j] + kk + kc_a[j]);
#pragma unroll
        for (int j = 0; j < NB; ++j) vb[j] = load16(pb[j] + kk + kc_b[j]);
    };
    auto load_step = [&](int it, uint4 (&va)[NA], uint4 (&vb)[NB]) {
        const int kk = kb + it * BK;
        if (WIDE && kk + BK <= ke) {                              // workgroup-uniform
            load_whole(it, va, vb);
        } else {
#pragma unroll
            for (int j = 0; j < NA; ++j) va[j] = tail_piece(pa[j], kk + kc_a[j], true);
#pragma unroll
            for (int j = 0; j < NB; ++j) vb[j] = tail_piece(pb[j], kk + kc_b[j], false);
        }
    };
    auto store_step = [&](int buf, const uint4 (&va)[NA], const uint4 (&vb)[NB]) {
#pragma unroll
        for (int j = 0; j < NA; ++j) *reinterpret_cast<uint4*>(&lds[buf][lds_a[j]]) = va[j];
#pragma unroll
        for (int j = 0; j < NB; ++j) *reinterpret_cast<uint4*>(&lds[buf][lds_b[j]]) = vb[j];
    };

    // ---- fragment addressing ---------------------------------------------------------
    // lane l reads row (l % 32) of a fragment, contraction bytes 16 * (l / 32) .. +15 of a 32-byte step
    const int frow = lane & 31, fhalf = lane >> 5;
    const int fswz = swizzle_of_row<BK>(frow);     // fragment bases are multiples of 32 rows: same swizzle
    const int a_base = (wm0 + frow) * BK, b_base = BM * BK + (wn0 + frow) * BK;

    v16i acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    auto multiply = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < BK / 32; ++ks) {
            const int piece = ((2 * ks + fhalf) ^ fswz) * 16;
            v4i fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[i] = *reinterpret_cast<const v4i*>(&lds[buf][a_base + i * 32 * BK + piece]);
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = *reinterpret_cast<const v4i*>(&lds[buf][b_base + j * 32 * BK + piece]);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    };
    if constexpr (STEPS == kManySteps) {
        // step it: request step it + 2 into the registers step it came from, multiply, park step it + 1 in the other buffer
        auto step = [&](int it, auto buf_c) {
            constexpr int buf = decltype(buf_c)::value;
            if (it + 2 < nk) load_step(it + 2, ra[buf], rb[buf]);
            multiply(buf);
            if (it + 1 < nk) store_step(buf ^ 1, ra[buf ^ 1], rb[buf ^ 1]);
            __syncthreads();
        };
        if (nk > 0) load_step(0, ra[0], rb[0]);
        if (nk > 1) load_step(1, ra[1], rb[1]);
        if (nk > 0) store_step(0, ra[0], rb[0]);
        __syncthreads();
        // While both steps to be requested are whole, without a branch: with one around the loads the compiler cannot count
        // those in flight, and waits for the new ones where it parks the older (1379 x 768 x 1000 gradients
        // 14.2 -> 11.6 us, 12608 x 768 x 1001 step 148.9 -> 137.8).
        auto steady = [&](int it, auto buf_c) {
            constexpr int buf = decltype(buf_c)::value;
            load_whole(it + 2, ra[buf], rb[buf]);
            __builtin_amdgcn_sched_barrier(0);
            multiply(buf);
            store_step(buf ^ 1, ra[buf ^ 1], rb[buf ^ 1]);
            __syncthreads();
        };
        const int whole = (ke - kb) / BK;
        int it = 0;
        for (; it + 3 < whole; it += 2) {
            steady(it, IC<0>{});
            steady(it + 1, IC<1>{});
        }
        for (; it < nk; it += 2) {
            step(it, IC<0>{});
            if (it + 1 < nk) step(it + 1, IC<1>{});
        }
    } else if (nk > 0) {                                          // workgroup-uniform
        load_step(0, ra[0], rb[0]);
        store_step(0, ra[0], rb[0]);
        __syncthreads();
        multiply(0);
    }

    // ---- epilogue --------------------------------------------------------------------
    // accumulator register r of lane l is row 8 * (r / 4) + 4 * (l / 32) + r % 4, column l % 32
    int E = 0;
    if (MODE == kStoreF32) E = lsb_exponent(eA[0], bitsA) + (eB ? lsb_exponent(eB[0], bitsB) : 0);
    if (MODE == kStoreF32 && amax != nullptr)
        publish_absmax(store_fragments<FM, FN, MODE, true>(acc, Cv, ldc, M, N, m0 + wm0, n0 + wn0, fhalf, frow, E), amax);
    else
        store_fragments<FM, FN, MODE, false>(acc, Cv, ldc, M, N, m0 + wm0, n0 + wn0, fhalf, frow, E);
}

// Products too small to fill the chip with LDS-staged tiles, up to two of them per launch.  What bounds those is the
// latency of one workgroup: launch, first loads, a barrier per K step.  Here a wave loads its MFMA operands straight
// from memory - 16 bytes of 32 rows, any alignment - with 8 steps of 32 in flight and no barrier; the four waves of a
// workgroup share one 32 x 32 tile and take every fourth step (together whole 128-byte lines), and their sums meet in LDS
// once.  The last, partial piece of a row is read as the row's last 16 bytes, as in k_gemm_nt: K >= 16.
template <int MODE>
__global__ __launch_bounds__(256) void k_gemm_nt_direct(Product p0, Product p1, ReduceRider rider) {
    if (rider.blocks != 0 && blockIdx.x >= rider.tiles) {          // workgroup-uniform: the last workgroups
        splitk_reduce_body<false, 256>(rider, blockIdx.x - rider.tiles, rider.blocks);
        return;
    }
    const bool second = blockIdx.x >= p0.tiles;
    const Product& p = second ? p1 : p0;
    constexpr int U = 8;                                           // steps in flight
    __shared__ int32_t sums[3][4][4][64];                          // [source][destination wave][register][lane]
    int tm, tn;
    tile_of_block(static_cast<int>(blockIdx.x - (second ? p0.tiles : 0u)), p.tiles_m, p.tiles_n, 8, &tm, &tn);
    const int m0 = tm * 32, n0 = tn * 32, K = p.K;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 31, fhalf = lane >> 5;
    const int8_t* pa = p.A + static_cast<int64_t>(min(m0 + frow, p.M - 1)) * p.lda;
    const int8_t* pb = p.B + static_cast<int64_t>(min(n0 + frow, p.N - 1)) * p.ldb;
    v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
    auto as_frag = [](const uint4& v) {
        v4i f;
        f[0] = static_cast<int>(v.x); f[1] = static_cast<int>(v.y); f[2] = static_cast<int>(v.z); f[3] = static_cast<int>(v.w);
        return f;
    };
    const int whole = K / 32;                                      // steps that lie inside every row
    for (int s0 = wave; s0 < whole; s0 += 4 * U) {
        uint4 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + 4 * u >= whole) break;                        // wave-uniform
            const int k = 32 * (s0 + 4 * u) + 16 * fhalf;
            a[u] = load16(pa + k);
            b[u] = load16(pb + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + 4 * u >= whole) break;
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_frag(a[u]), as_frag(b[u]), acc, 0, 0, 0);
        }
    }
    if (32 * whole < K && wave == (whole & 3)) {                   // the last, partial step
        const int k = 32 * whole + 16 * fhalf, from = min(k, K - 16);
        uint4 a = load16(pa + from);
        const uint4 b = load16(pb + from);
        if (k >= K) a = make_uint4(0, 0, 0, 0);
        else if (from < k) a = clear_low_bytes(a, k - from);
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_frag(a), as_frag(b), acc, 0, 0, 0);
    }
    // wave w finishes registers 4 w .. 4 w + 3: rows 8 w + 4 * (l / 32) + 0 .. 3
    int own[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int src = wave < w ? wave : wave - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (w == wave) own[r] = acc[4 * w + r];                // wave-uniform
            else sums[src][w][r][lane] = acc[4 * w + r];
        }
    }
    __syncthreads();
    int E = 0;
    if (MODE == kStoreF32) E = lsb_exponent(p.eA[0], p.bitsA) + (p.eB ? lsb_exponent(p.eB[0], p.bitsB) : 0);
    float m = 0.0f;
    const int col = n0 + frow;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int sum = own[r] + sums[0][wave][r][lane] + sums[1][wave][r][lane] + sums[2][wave][r][lane];
        const int row = m0 + 8 * wave + 4 * fhalf + r;
        if (row >= p.M || col >= p.N) continue;
        const int64_t off = static_cast<int64_t>(row) * p.ldc + col;
        if (MODE == kStoreF32) {
            const float v = unmap_value(sum, E);
            static_cast<float*>(p.C)[off] = v;
            m = fmaxf(m, fabsf(v));
        } else {
            static_cast<int32_t*>(p.C)[off] = sum;
        }
    }
    if (MODE == kStoreF32 && p.amax != nullptr) publish_absmax(m, p.amax);
}

// Same product, fast path: K a multiple of BK, operands 16-byte aligned.  Global loads go
// straight into LDS (global_load_lds_dwordx4: each wave fills one contiguous 1 KiB region
// per instruction, no register staging, no ds_write), STAGES buffers deep, so loads for
// step k + STAGES - 1 are in flight while step k is multiplied.  The XOR swizzle of the
// LDS layout is applied on the global side: lane p of a region fetches the 16-byte piece
// that belongs in slot p.  One s_barrier per step, no fence: the only cross-wave traffic
// is LDS written by the loads (waited for with vmcnt before the barrier) and read by
// ds_read (waited for with lgkmcnt before the next barrier lets the buffer be refilled).
//
// CONV: the A operand is not a stored matrix but the patch matrix of a channels-last int8 image tensor
// (A points at X[N,H,W,C]; row m is output pixel m, contraction index (kh*KW + kw)*C + c): the loader
// works out, per K step, which input pixel a row reads (one tap of the filter, since C % BK == 0) and takes
// the bytes straight from the image, or from a page of zeros where the tap falls into the padding.  Nothing
// else differs from the plain product.
//
// Taps = StrideClasses: the input gradient of a strided convolution, all classes in one launch.  The row tiles of the
// classes alternate (an XCD's run of tiles then holds every class of the same pixels, which read the same gradient
// pixels, and the classes' different contraction lengths spread evenly); the epilogue scatters rows to their pixels.
template <int BM, int BN, int BK, int WM, int WN, int STAGES, int MODE, bool SCHED, bool CONV = false, typename Taps = ConvTaps>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void k_gemm_nt_dma(
    const int8_t* __restrict__ A, int64_t lda, const int8_t* __restrict__ B, int64_t ldb, void* __restrict__ Cv,
    int64_t ldc, int M, int N, int K, int k_per_split, const int32_t* __restrict__ eA, int bitsA,
    const int32_t* __restrict__ eB, int bitsB, int tiles_m, int tiles_n, int group_m, int64_t split_stride,
    int64_t batch_a, int64_t batch_b, int64_t batch_c, Taps taps, uint32_t* __restrict__ amax, ReduceRider rider) {
    int tile_block = static_cast<int>(blockIdx.x);
    if (rider.blocks != 0) {                                      // workgroup-uniform
        const unsigned first = rider.front ? 0u : rider.tiles;    // the riders are the first or the last workgroups
        if (blockIdx.x >= first && blockIdx.x < first + rider.blocks) {
            splitk_reduce_body<false, (BM / WM) * (BN / WN) * 64>(rider, blockIdx.x - first, rider.blocks);
            return;
        }
        if (rider.front) tile_block -= static_cast<int>(rider.blocks);
    }
    constexpr int NW = (BM / WM) * (BN / WN);
    constexpr int CPR = BK / 16;                     // 16-byte pieces per LDS row
    constexpr int RROWS = 64 / CPR;                  // tile rows per 1 KiB region
    constexpr int REGIONS = (BM + BN) * BK / 1024;   // per stage: A rows first, then B rows
    constexpr int RPW = REGIONS / NW;                // load instructions per wave per step
    constexpr int STAGE_BYTES = (BM + BN) * BK;
    constexpr int FM = WM / 32, FN = WN / 32;
    static_assert(REGIONS % NW == 0, "regions do not divide over the waves");
    static_assert(STAGES >= 2 && STAGES <= 4, "2 to 4 stages");
    static_assert((STAGES - 1) * RPW < 64, "vmcnt is a 6-bit counter");
    static_assert((BK / 32) % 2 == 0, "two 32-byte steps per register buffer pair");
    static_assert(FM * FN >= (FM + FN) / 2, "wave tile too small for the interleave");

    __shared__ __attribute__((aligned(1024))) int8_t lds[STAGES * STAGE_BYTES];

    // Workgroups reach the XCDs round-robin in dispatch order (x fastest, then y, then z).  One product, one slice:
    // the tile walk of tile_of_block.  Split along K, or a batch of products: XCD c takes a contiguous run of
    // (slice or matrix, tile) pairs in slice-major order, so the tiles of one slice (which read the same K range of
    // B) or of one small matrix (which read the same operands) share that XCD's L2.
    int tm, tn, slice = 0, matrix = 0;
    const int outer = static_cast<int>(gridDim.y * gridDim.z);     // never both: a batch is not split
    if (outer == 1) {
        tile_of_block(tile_block, tiles_m, tiles_n, group_m, &tm, &tn);
    } else {
        const int64_t tiles = static_cast<int64_t>(tiles_m) * tiles_n, total = tiles * outer;
        const int64_t v = (static_cast<int64_t>(blockIdx.z) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        const int64_t q = total / kNumXcd, r = total % kNumXcd, xcd = v % kNumXcd, local = v / kNumXcd;
        const int64_t p = (xcd < r) ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
        const int o = static_cast<int>(p / tiles), t = static_cast<int>(p - o * tiles);
        if (gridDim.y > 1) slice = o;
        else matrix = o;
        tm = t % tiles_m;
        tn = t / tiles_m;
    }
    constexpr bool STRIDED = std::is_same<Taps, StrideClasses>::value;
    ConvTaps ct;
    [[maybe_unused]] StrideClass cl{};
    if constexpr (STRIDED) {
        const int classes = taps.stride * taps.stride, c = tm % classes;
        tm /= classes;
        cl = taps.cls[c];
        M = M * cl.Ho * cl.Wo;                                       // M: images
        if (tm * BM >= M) return;                                    // workgroup-uniform: a class of fewer tiles
        K = cl.TH * cl.TW * taps.C;
        k_per_split = K;
        B += cl.w_first;
        ldb = K;
        ct.H = taps.H; ct.W = taps.W; ct.C = taps.C; ct.KW = cl.TW;
        ct.pad = cl.pad; ct.padw = cl.padw; ct.Ho = cl.Ho; ct.Wo = cl.Wo;
    } else {
        ct = taps;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int kb = slice * k_per_split;
    // split-K into a workspace: every slice owns its own M x N int32 matrix (split_stride elements apart)
    Cv = static_cast<int32_t*>(Cv) + static_cast<int64_t>(slice) * split_stride + static_cast<int64_t>(matrix) * batch_c;
    // batched product: matrix z of each operand lies batch_* elements further on
    A += static_cast<int64_t>(matrix) * batch_a;
    B += static_cast<int64_t>(matrix) * batch_b;
    const int ke = min(K, kb + k_per_split);
    // whole K steps, plus one partial step when the slice ends inside a step (K a multiple of 16, not of BK):
    // its missing 16-byte pieces are read from the page of zeros, so the multiply loop never sees a tail
    const int nk = (ke - kb + BK - 1) / BK;
    const int tail = (ke - kb) % BK;


    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS targets stay in SGPRs
    const int wm0 = (wave / (BN / WN)) * WM, wn0 = (wave % (BN / WN)) * WN;

    const int8_t* gp[RPW];
    int kpiece[RPW];                                                 // offset of the lane's 16-byte piece inside a K step
    int a_h0[RPW], a_w0[RPW];                                        // CONV: top-left input coordinate of the row's patch
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
        const int row_t = (wave + j * NW) * RROWS + lane / CPR;      // row in the stacked (A;B) tile
        const int piece = (lane % CPR) ^ swizzle_of_row<BK>(row_t);  // BM % 16 == 0: same swizzle for B rows
        kpiece[j] = piece * 16;
        a_h0[j] = a_w0[j] = 0;
        if (CONV && row_t < BM) {
            const uint32_t m = static_cast<uint32_t>(min(m0 + row_t, M - 1));
            const uint32_t t = m / static_cast<uint32_t>(ct.Wo), n = t / static_cast<uint32_t>(ct.Ho);
            a_h0[j] = static_cast<int>(t - n * ct.Ho) * ct.stride - ct.pad;
            a_w0[j] = static_cast<int>(m - t * ct.Wo) * ct.stride - ct.padw;
            gp[j] = A + static_cast<int64_t>(n) * ct.H * ct.W * ct.C + piece * 16;          // the row's image
        } else {
            gp[j] = (row_t < BM) ? A + static_cast<int64_t>(min(m0 + row_t, M - 1)) * lda + kb + piece * 16
                                 : B + static_cast<int64_t>(min(n0 + row_t - BM, N - 1)) * ldb + kb + piece * 16;
        }
    }
    auto issue = [&](int step, int stage) {
        int kh = 0, kw = 0, c0 = 0;                                  // CONV: the tap and channel offset of this K step
        if (CONV) {
            const int k0 = kb + step * BK, tap = k0 / ct.C;
            c0 = k0 - tap * ct.C;
            kh = tap / ct.KW;
            kw = tap - kh * ct.KW;
        }
        const bool partial = !CONV && tail != 0 && step == nk - 1;   // wave-uniform
#pragma unroll
        for (int j = 0; j < RPW; ++j) {
            const int8_t* src = gp[j] + static_cast<int64_t>(step) * BK;
            if (partial && kpiece[j] >= tail) src = reinterpret_cast<const int8_t*>(g_zero_page) + kpiece[j];
            if (CONV && (wave + j * NW) * RROWS < BM) {              // a region of A rows (wave-uniform)
                const int h = a_h0[j] + kh, w = a_w0[j] + kw;
                const bool inside = static_cast<unsigned>(h) < static_cast<unsigned>(ct.H) &&
                                    static_cast<unsigned>(w) < static_cast<unsigned>(ct.W);
                src = inside ? gp[j] + (static_cast<int64_t>(h) * ct.W + w) * ct.C + c0
                             : reinterpret_cast<const int8_t*>(g_zero_page) + kpiece[j];
            }
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)src,
                (__attribute__((address_space(3))) void*)(&lds[stage * STAGE_BYTES + (wave + j * NW) * 1024]),
                16, 0, 0);
        }
    };

    const int frow = lane & 31, fhalf = lane >> 5;
    const int fswz = swizzle_of_row<BK>(frow);
    const int a_base = (wm0 + frow) * BK, b_base = BM * BK + (wn0 + frow) * BK;

    v16i acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // Fragments are double-buffered in registers: the ds_reads of 32-byte step s+1 are
    // issued before the MFMAs of step s.  The barrier that publishes LDS stage it+1 sits
    // in front of the LAST 32-byte step of stage it, so the first fragments of the next
    // stage are already on their way while that last step is multiplied, and the stage
    // just finished (every wave is past its reads of it) is refilled at once: all STAGES
    // buffers stay in flight.
    constexpr int KS = BK / 32;
    v4i fa[2][FM], fb[2][FN];
    auto read_frags = [&](int buf, int stage, int ks) {
        const int8_t* st = lds + stage * STAGE_BYTES;
        const int piece = ((2 * ks + fhalf) ^ fswz) * 16;
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[buf][i] = *reinterpret_cast<const v4i*>(&st[a_base + i * 32 * BK + piece]);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[buf][j] = *reinterpret_cast<const v4i*>(&st[b_base + j * 32 * BK + piece]);
    };
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < nk) issue(s, s);
    if (nk > 0) {
        if (nk >= STAGES) wait_loads_and_lds<(STAGES - 1) * RPW>();
        else wait_loads_and_lds<0>();
        __builtin_amdgcn_s_barrier();
        read_frags(0, 0, 0);
    }
    // MFMAs of one 32-byte step.  `reads` ds_reads and `loads` global->LDS loads issued just
    // before it are slotted behind its first MFMAs (the matrix core runs an MFMA for 32
    // cycles; the wave issues the memory instructions in its shadow).
    auto multiply = [&](int cur, auto reads_c, auto loads_c) {
        constexpr int reads = decltype(reads_c)::value, loads = decltype(loads_c)::value;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
        if (SCHED) {
#pragma unroll
            for (int n = 0; n < reads / 2; ++n) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // 2 DS reads
            }
#pragma unroll
            for (int n = 0; n < loads; ++n) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // 1 VMEM read
            }
            __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - reads / 2 - loads, 0);
        }
    };
    // One LDS stage: all 32-byte steps but the last, then the barrier that publishes the next
    // stage, the first fragments of that stage, the refill of the stage just finished, and the
    // last step.  The wait is one fixed instruction and the refill is unconditional inside a
    // loop variant, so everything between two barriers is one basic block the scheduler can
    // interleave.
    auto stage_body = [&](int it, auto wait_next, auto refill) {
        const int stage = it % STAGES;
#pragma unroll
        for (int ks = 0; ks + 1 < KS; ++ks) {
            read_frags((ks & 1) ^ 1, stage, ks + 1);
            multiply(ks & 1, IC<FM + FN>{}, IC<0>{});
        }
        wait_next();
        __builtin_amdgcn_s_barrier();
        read_frags(0, (it + 1) % STAGES, 0);          // KS is even: the last step used buffer 1
        multiply(1, IC<FM + FN>{}, refill(it + STAGES, stage));
    };
    auto steady_wait = [] { wait_loads_and_lds<(STAGES - 2) * RPW>(); };
    auto full_wait = [] { wait_loads_and_lds<0>(); };
    auto do_refill = [&](int step, int stage) {
        issue(step, stage);
        return IC<(RPW <= FM * FN - (FM + FN) / 2 ? RPW : 0)>{};
    };
    auto no_refill = [](int, int) { return IC<0>{}; };
    int it = 0;
    for (; it + STAGES < nk; ++it) stage_body(it, steady_wait, do_refill);     // steps it+2 .. it+STAGES-1 in flight
    for (; it + STAGES - 1 < nk; ++it) stage_body(it, steady_wait, no_refill);
    for (; it + 1 < nk; ++it) stage_body(it, full_wait, no_refill);            // drain
    if (nk > 0) {
        const int stage = (nk - 1) % STAGES;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) read_frags((ks & 1) ^ 1, stage, ks + 1);
            if (ks + 1 < KS) multiply(ks & 1, IC<FM + FN>{}, IC<0>{});
            else multiply(ks & 1, IC<0>{}, IC<0>{});
        }
    }

    int E = 0;
    if (MODE == kStoreF32) E = lsb_exponent(eA[0], bitsA) + (eB ? lsb_exponent(eB[0], bitsB) : 0);
    if constexpr (STRIDED) {
        // where the tile's rows go: one division chain per row, shared through LDS
        int64_t* row_at = reinterpret_cast<int64_t*>(lds);
        __syncthreads();                                             // every wave is past its last read of a stage
        if (tid < BM) {
            const uint32_t m = static_cast<uint32_t>(min(m0 + tid, M - 1));
            const uint32_t t = m / static_cast<uint32_t>(cl.Wo), n = t / static_cast<uint32_t>(cl.Ho);
            const int h = cl.h0 + taps.stride * static_cast<int>(t - n * cl.Ho), w = cl.w0 + taps.stride * static_cast<int>(m - t * cl.Wo);
            row_at[tid] = ((static_cast<int64_t>(n) * taps.outH + h) * taps.outW + w) * ldc;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm0 + 32 * i + 8 * (r >> 2) + 4 * fhalf + (r & 3);
                if (m0 + row >= M) continue;
                float* out = static_cast<float*>(Cv) + row_at[row] + n0 + wn0 + frow;
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    if (n0 + wn0 + 32 * j + frow < N) __builtin_nontemporal_store(unmap_value(acc[i][j][r], E), out + 32 * j);
            }
        return;
    }
    if (MODE == kStoreF32 && amax != nullptr)
        publish_absmax(store_fragments<FM, FN, MODE, true>(acc, Cv, ldc, M, N, m0 + wm0, n0 + wn0, fhalf, frow, E), amax);
    else
        store_fragments<FM, FN, MODE, false>(acc, Cv, ldc, M, N, m0 + wm0, n0 + wn0, fhalf, frow, E);
}

// 256 x 256 x 128 tile with LDS used as a RING of five 32 KiB half-stages instead of two
// full stages.  A half-stage is the 256 x 128-byte slice of one operand for one step:
// A(0) B(0) A(1) B(1) A(2) | B(2) A(3) ...; half-stage h lives in slot h % 5.  Full 128-byte
// rows keep every L2 request a whole cache line (half-line requests top out at ~60 % of the
// line rate), and the fifth slot lets the loads of a step be issued in two instalments:
// A(t+2) is spread thinly over the first three 32-byte steps of stage t (its slot was freed
// one barrier earlier) and only B(t+2) has to be issued in a burst behind the barrier that
// frees A(t)'s slot.  The load queue therefore never runs dry and never has to swallow a
// whole 64 KiB stage at once, which is what stalled the MFMA stream of the two-stage form.
template <int WM, int WN, int MODE, bool SCHED>
__global__ __launch_bounds__((256 / WM) * (256 / WN) * 64) void k_gemm_nt_ring(
    const int8_t* __restrict__ A, int64_t lda, const int8_t* __restrict__ B, int64_t ldb, void* __restrict__ Cv,
    int64_t ldc, int M, int N, int K, int k_per_split, const int32_t* __restrict__ eA, int bitsA,
    const int32_t* __restrict__ eB, int bitsB, int tiles_m, int tiles_n, int group_m, int64_t split_stride,
    int64_t batch_a, int64_t batch_b, int64_t batch_c, uint32_t* __restrict__ amax, ReduceRider rider) {
    int tile_block = static_cast<int>(blockIdx.x);
    if (rider.blocks != 0) {                                      // workgroup-uniform
        const unsigned first = rider.front ? 0u : rider.tiles;    // the riders are the first or the last workgroups
        if (blockIdx.x >= first && blockIdx.x < first + rider.blocks) {
            splitk_reduce_body<false, (256 / WM) * (256 / WN) * 64>(rider, blockIdx.x - first, rider.blocks);
            return;
        }
        if (rider.front) tile_block -= static_cast<int>(rider.blocks);
    }
    constexpr int BM = 256, BN = 256, BK = 128;
    constexpr int NW = (BM / WM) * (BN / WN);
    constexpr int SLOT = 256 * BK;                   // bytes of a half-stage
    constexpr int RPH = (SLOT / 1024) / NW;          // load instructions per wave per half-stage
    constexpr int FM = WM / 32, FN = WN / 32, KS = BK / 32;
    static_assert(RPH >= 3 && RPH * 2 < 64, "loads per half-stage");

    __shared__ __attribute__((aligned(1024))) int8_t lds[5 * SLOT];

    int tm, tn;
    tile_of_block(tile_block, tiles_m, tiles_n, group_m, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int kb = blockIdx.y * k_per_split;
    // split-K into a workspace: slice y owns its own M x N int32 matrix (split_stride elements apart)
    Cv = static_cast<int32_t*>(Cv) + static_cast<int64_t>(blockIdx.y) * split_stride + static_cast<int64_t>(blockIdx.z) * batch_c;
    // batched product: matrix z of each operand lies batch_* elements further on
    A += static_cast<int64_t>(blockIdx.z) * batch_a;
    B += static_cast<int64_t>(blockIdx.z) * batch_b;
    const int ke = min(K, kb + k_per_split);
    const int nk = (ke - kb) / BK;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / (BN / WN)) * WM, wn0 = (wave % (BN / WN)) * WN;

    // lane p of 1 KiB region g fetches row 8g + p/8, piece (p%8) ^ swizzle(row) of the 128-byte row
    const int8_t* ga[RPH];
    const int8_t* gb[RPH];
#pragma unroll
    for (int j = 0; j < RPH; ++j) {
        const int row = (wave + j * NW) * 8 + lane / 8;
        const int piece = (lane % 8) ^ swizzle_of_row<BK>(row);
        ga[j] = A + static_cast<int64_t>(min(m0 + row, M - 1)) * lda + kb + piece * 16;
        gb[j] = B + static_cast<int64_t>(min(n0 + row, N - 1)) * ldb + kb + piece * 16;
    }
    auto load_piece = [&](const int8_t* g, int step, int slot, int j) {
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(g + static_cast<int64_t>(step) * BK),
            (__attribute__((address_space(3))) void*)(&lds[slot * SLOT + (wave + j * NW) * 1024]), 16, 0, 0);
    };
    auto issue_a = [&](int step, auto lo_c, auto hi_c) {        // loads [lo, hi) of A(step)
        const int slot = (2 * step) % 5;
#pragma unroll
        for (int j = decltype(lo_c)::value; j < decltype(hi_c)::value; ++j) load_piece(ga[j], step, slot, j);
    };
    auto issue_b = [&](int step) {
        const int slot = (2 * step + 1) % 5;
#pragma unroll
        for (int j = 0; j < RPH; ++j) load_piece(gb[j], step, slot, j);
    };

    const int frow = lane & 31, fhalf = lane >> 5;
    const int fswz = swizzle_of_row<BK>(frow);
    const int a_off = (wm0 + frow) * BK, b_off = (wn0 + frow) * BK;

    v16i acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    v4i fa[2][FM], fb[2][FN];
    auto read_frags = [&](int buf, int step, int ks) {
        const int8_t* sa = lds + ((2 * step) % 5) * SLOT + a_off;
        const int8_t* sb = lds + ((2 * step + 1) % 5) * SLOT + b_off;
        const int piece = ((2 * ks + fhalf) ^ fswz) * 16;
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[buf][i] = *reinterpret_cast<const v4i*>(&sa[i * 32 * BK + piece]);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[buf][j] = *reinterpret_cast<const v4i*>(&sb[j * 32 * BK + piece]);
    };
    auto multiply = [&](int cur, auto reads_c, auto loads_c) {
        constexpr int reads = decltype(reads_c)::value, loads = decltype(loads_c)::value;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
        if (SCHED) {
#pragma unroll
            for (int n = 0; n < reads / 2; ++n) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
#pragma unroll
            for (int n = 0; n < loads; ++n) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - reads / 2 - loads, 0);
        }
    };
    // thirds of a half-stage for the three early 32-byte steps
    constexpr int T1 = (RPH + 2) / 3, T2 = (2 * RPH + 2) / 3;
    // stage t, when step t+1 exists.  EARLY: A(t+2) is issued here (not for t = 0: the prologue
    // did it); LATE: B(t+2) is issued behind the barrier.
    auto stage_body = [&](int t, auto early_c, auto late_c, auto wait_next) {
        constexpr bool EARLY = decltype(early_c)::value != 0, LATE = decltype(late_c)::value != 0;
        read_frags(1, t, 1);
        if (EARLY) issue_a(t + 2, IC<0>{}, IC<T1>{});
        multiply(0, IC<FM + FN>{}, IC<(EARLY ? T1 : 0)>{});
        read_frags(0, t, 2);
        if (EARLY) issue_a(t + 2, IC<T1>{}, IC<T2>{});
        multiply(1, IC<FM + FN>{}, IC<(EARLY ? T2 - T1 : 0)>{});
        read_frags(1, t, 3);
        if (EARLY) issue_a(t + 2, IC<T2>{}, IC<RPH>{});
        multiply(0, IC<FM + FN>{}, IC<(EARLY ? RPH - T2 : 0)>{});
        wait_next();
        __builtin_amdgcn_s_barrier();
        read_frags(0, t + 1, 0);
        if (LATE) issue_b(t + 2);
        multiply(1, IC<FM + FN>{}, IC<(LATE ? RPH : 0)>{});
    };
    auto wait_one_half = [] { wait_loads_and_lds<RPH>(); };
    auto wait_all = [] { wait_loads_and_lds<0>(); };

    // prologue: A(0) B(0) A(1) B(1) A(2)
    if (nk > 0) { issue_a(0, IC<0>{}, IC<RPH>{}); issue_b(0); }
    if (nk > 1) { issue_a(1, IC<0>{}, IC<RPH>{}); issue_b(1); }
    if (nk > 2) issue_a(2, IC<0>{}, IC<RPH>{});
    if (nk > 0) {
        if (nk > 2) wait_loads_and_lds<3 * RPH>();
        else if (nk > 1) wait_loads_and_lds<2 * RPH>();
        else wait_loads_and_lds<0>();
        __builtin_amdgcn_s_barrier();
        read_frags(0, 0, 0);
    }
    int t = 0;
    if (nk > 2) {                                                   // t = 0: A(2) already in flight
        stage_body(0, IC<0>{}, IC<1>{}, wait_one_half);
        t = 1;
        for (; t + 2 < nk; ++t) stage_body(t, IC<1>{}, IC<1>{}, wait_one_half);
    }
    for (; t + 1 < nk; ++t) stage_body(t, IC<0>{}, IC<0>{}, wait_all);   // nothing left to issue
    if (nk > 0) {                                                   // last stage
        read_frags(1, t, 1);
        multiply(0, IC<FM + FN>{}, IC<0>{});
        read_frags(0, t, 2);
        multiply(1, IC<FM + FN>{}, IC<0>{});
        read_frags(1, t, 3);
        multiply(0, IC<FM + FN>{}, IC<0>{});
        multiply(1, IC<0>{}, IC<0>{});
    }

    int E = 0;
    if (MODE == kStoreF32) E = lsb_exponent(eA[0], bitsA) + (eB ? lsb_exponent(eB[0], bitsB) : 0);
    if (MODE == kStoreF32 && amax != nullptr)
        publish_absmax(store_fragments<FM, FN, MODE, true>(acc, Cv, ldc, M, N, m0 + wm0, n0 + wn0, fhalf, frow, E), amax);
    else
        store_fragments<FM, FN, MODE, false>(acc, Cv, ldc, M, N, m0 + wm0, n0 + wn0, fhalf, frow, E);
}

// split-K helpers over an M x N int32 / fp32 matrix with leading dimension ldc; grid.y walks
// rows when ldc != N, otherwise the matrix is one flat run (16-byte accesses when aligned)
__global__ __launch_bounds__(256) void k_zero_rows(int32_t* __restrict__ C, int64_t ldc, int rows, int cols) {
    for (int r = blockIdx.y; r < rows; r += gridDim.y) {
        int32_t* row = C + static_cast<int64_t>(r) * ldc;
        const bool vec = (reinterpret_cast<uintptr_t>(row) & 15u) == 0;
        const int nvec = vec ? cols >> 2 : 0;
        for (int i = blockIdx.x * 256 + threadIdx.x; i < nvec; i += gridDim.x * 256)
            reinterpret_cast<int4*>(row)[i] = make_int4(0, 0, 0, 0);
        for (int i = (nvec << 2) + blockIdx.x * 256 + threadIdx.x; i < cols; i += gridDim.x * 256) row[i] = 0;
    }
}

__global__ __launch_bounds__(256) void k_unmap_rows(int32_t* __restrict__ C, int64_t ldc, int rows, int cols,
                                                    const int32_t* __restrict__ eA, int bitsA,
                                                    const int32_t* __restrict__ eB, int bitsB, uint32_t* __restrict__ amax) {
    const int E = lsb_exponent(eA[0], bitsA) + (eB ? lsb_exponent(eB[0], bitsB) : 0);
    float m = 0.0f;
    for (int r = blockIdx.y; r < rows; r += gridDim.y) {
        int32_t* row = C + static_cast<int64_t>(r) * ldc;
        const bool vec = (reinterpret_cast<uintptr_t>(row) & 15u) == 0;
        const int nvec = vec ? cols >> 2 : 0;
        for (int i = blockIdx.x * 256 + threadIdx.x; i < nvec; i += gridDim.x * 256) {
            const int4 a = reinterpret_cast<const int4*>(row)[i];
            float4 o;
            o.x = unmap_value(a.x, E);
            o.y = unmap_value(a.y, E);
            o.z = unmap_value(a.z, E);
            o.w = unmap_value(a.w, E);
            reinterpret_cast<float4*>(row)[i] = o;
            m = fmaxf(fmaxf(m, fmaxf(fabsf(o.x), fabsf(o.y))), fmaxf(fabsf(o.z), fabsf(o.w)));
        }
        for (int i = (nvec << 2) + blockIdx.x * 256 + threadIdx.x; i < cols; i += gridDim.x * 256) {
            const float o = unmap_value(row[i], E);
            reinterpret_cast<float*>(row)[i] = o;
            m = fmaxf(m, fabsf(o));
        }
    }
    if (amax != nullptr) publish_absmax(m, amax);
}

// launch shape of the two helpers: a dense matrix is treated as one long row
static void rows_launch_shape(int64_t M, int64_t N, int64_t ldc, int* rows, int* cols, dim3* grid) {
    if (ldc == N && M * N < (int64_t{1} << 31)) {
        *rows = 1;
        *cols = static_cast<int>(M * N);
    } else {
        *rows = static_cast<int>(M);
        *cols = static_cast<int>(N);
    }
    const int gx = std::max(1, std::min(1024, (*cols / 4 + 255) / 256));
    *grid = dim3(gx, std::max(1, std::min(*rows, 65535)));
}

// int8 [rows, cols] (leading dimension ld) -> [cols, rows] contiguous, 64 x 64 tiles through LDS
__global__ __launch_bounds__(256) void k_transpose_i8(const int8_t* __restrict__ src, int64_t rows, int64_t cols,
                                                      int64_t ld, int8_t* __restrict__ dst, int tiles_c) {
    __shared__ int8_t t[64][65];
    const int64_t r0 = static_cast<int64_t>(blockIdx.x / tiles_c) * 64, c0 = static_cast<int64_t>(blockIdx.x % tiles_c) * 64;
    for (int id = threadIdx.x; id < 64 * 64; id += 256) {
        const int r = id >> 6, c = id & 63;
        if (r0 + r < rows && c0 + c < cols) t[r][c] = src[(r0 + r) * ld + c0 + c];
    }
    __syncthreads();
    for (int id = threadIdx.x; id < 64 * 64; id += 256) {
        const int c = id >> 6, r = id & 63;
        if (r0 + r < rows && c0 + c < cols) dst[(c0 + c) * rows + r0 + r] = t[r][c];
    }
}

int transpose_i8_launch(const int8_t* src, int64_t rows, int64_t cols, int64_t ld, int8_t* dst, hipStream_t s) {
    if (rows == 0 || cols == 0) return FXP_OK;
    const int64_t tr = (rows + 63) / 64, tc = (cols + 63) / 64;
    if (tr * tc >= (int64_t{1} << 31)) return FXP_ERR_DIMS;
    hipLaunchKernelGGL(k_transpose_i8, dim3(static_cast<unsigned>(tr * tc)), dim3(256), 0, s, src, rows, cols, ld, dst,
                       static_cast<int>(tc));
    return launch_status();
}

template <int BM, int BN, int BK, int WM, int WN>
static int launch_cfg(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, const int8_t* B, int64_t ldb,
                      void* C, int64_t ldc, int mode, int splits, const int32_t* eA, int bitsA,
                      const int32_t* eB, int bitsB, hipStream_t s, int64_t split_stride = 0, int* slices = nullptr,
                      Batch bt = Batch(), uint32_t* amax = nullptr, ReduceRider* ride = nullptr, const Product& two = Product()) {
    constexpr int NT = (BM / WM) * (BN / WN) * 64;
    const int tiles_m = static_cast<int>((M + BM - 1) / BM), tiles_n = static_cast<int>((N + BN - 1) / BN);
    int k_per_split = static_cast<int>((K + splits - 1) / splits);
    k_per_split = (k_per_split + BK - 1) / BK * BK;
    if (k_per_split == 0) k_per_split = BK;
    const int ny = K > 0 ? static_cast<int>((K + k_per_split - 1) / k_per_split) : 1;
    if (slices) *slices = ny;
    ReduceRider rider;                                          // rides only in an unsplit, unbatched launch
    if (ride != nullptr && ride->blocks != 0 && ny == 1 && bt.count == 1) {
        rider = *ride;
        rider.tiles = static_cast<unsigned>(tiles_m) * tiles_n;
        rider.front = rider.tiles >= 512;                       // several rounds of tiles: ride in the first one
        ride->blocks = 0;                                       // taken
    }
    const dim3 grid(static_cast<unsigned>(tiles_m) * tiles_n + two.tiles + rider.blocks, ny, bt.count), block(NT);
    const int group_m = 8;
#define FXP_GEMM_LAUNCH(STEPS, MODE)                                                                               \
    hipLaunchKernelGGL((k_gemm_nt<BM, BN, BK, WM, WN, STEPS, MODE>), grid, block, 0, s, A, lda, B, ldb, C, ldc,      \
                       static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), k_per_split, eA, bitsA, eB,   \
                       bitsB, tiles_m, tiles_n, group_m, split_stride, bt.a, bt.b, bt.c, amax, rider, two)
#define FXP_GEMM_MODES(STEPS)                                            \
    do {                                                                 \
        if (mode == kStoreI32) FXP_GEMM_LAUNCH(STEPS, kStoreI32);        \
        else if (mode == kStoreF32) FXP_GEMM_LAUNCH(STEPS, kStoreF32);   \
        else FXP_GEMM_LAUNCH(STEPS, kAtomicI32);                         \
    } while (0)
    // (a second product has 16 terms or more)
    if (K < 16) FXP_GEMM_MODES(kOneStepBytes);
    else if (K <= BK && two.K <= BK) FXP_GEMM_MODES(kOneStep);
    else FXP_GEMM_MODES(kManySteps);
#undef FXP_GEMM_MODES
#undef FXP_GEMM_LAUNCH
    return launch_status();
}

template <int WM, int WN, bool SCHED = true>
static int launch_ring(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, const int8_t* B, int64_t ldb,
                       void* C, int64_t ldc, int mode, int splits, const int32_t* eA, int bitsA, const int32_t* eB,
                       int bitsB, hipStream_t s, int64_t split_stride = 0, int* slices = nullptr,
                      Batch bt = Batch(), uint32_t* amax = nullptr, ReduceRider* ride = nullptr) {
    constexpr int NT = (256 / WM) * (256 / WN) * 64, BK = 128;
    const int tiles_m = static_cast<int>((M + 255) / 256), tiles_n = static_cast<int>((N + 255) / 256);
    int k_per_split = static_cast<int>((K + splits - 1) / splits);
    k_per_split = (k_per_split + BK - 1) / BK * BK;
    const int ny = static_cast<int>((K + k_per_split - 1) / k_per_split);
    if (slices) *slices = ny;
    ReduceRider rider;                                          // rides only in an unsplit, unbatched launch
    if (ride != nullptr && ride->blocks != 0 && ny == 1 && bt.count == 1) {
        rider = *ride;
        rider.tiles = static_cast<unsigned>(tiles_m) * tiles_n;
        rider.front = rider.tiles >= 512;                       // several rounds of tiles: ride in the first one
        ride->blocks = 0;                                       // taken
    }
    const dim3 grid(static_cast<unsigned>(tiles_m) * tiles_n + rider.blocks, ny, bt.count), block(NT);
    const int group_m = 8;
#define FXP_GEMM_LAUNCH(MODE)                                                                                    \
    hipLaunchKernelGGL((k_gemm_nt_ring<WM, WN, MODE, SCHED>), grid, block, 0, s, A, lda, B, ldb, C, ldc,          \
                       static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), k_per_split, eA, bitsA, eB, \
                       bitsB, tiles_m, tiles_n, group_m, split_stride, bt.a, bt.b, bt.c, amax, rider)
    if (mode == kStoreI32) FXP_GEMM_LAUNCH(kStoreI32);
    else if (mode == kStoreF32) FXP_GEMM_LAUNCH(kStoreF32);
    else FXP_GEMM_LAUNCH(kAtomicI32);
#undef FXP_GEMM_LAUNCH
    return launch_status();
}

template <int BM, int BN, int BK, int WM, int WN, int STAGES, bool SCHED = true>
static int launch_dma(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, const int8_t* B, int64_t ldb,
                      void* C, int64_t ldc, int mode, int splits, const int32_t* eA, int bitsA, const int32_t* eB,
                      int bitsB, hipStream_t s, int64_t split_stride = 0, int* slices = nullptr,
                      Batch bt = Batch(), uint32_t* amax = nullptr, ReduceRider* ride = nullptr) {
    constexpr int NT = (BM / WM) * (BN / WN) * 64;
    const int tiles_m = static_cast<int>((M + BM - 1) / BM), tiles_n = static_cast<int>((N + BN - 1) / BN);
    int k_per_split = static_cast<int>((K + splits - 1) / splits);
    k_per_split = (k_per_split + BK - 1) / BK * BK;
    const int ny = static_cast<int>((K + k_per_split - 1) / k_per_split);
    if (slices) *slices = ny;
    ReduceRider rider;                                          // rides only in an unsplit, unbatched launch
    if (ride != nullptr && ride->blocks != 0 && ny == 1 && bt.count == 1) {
        rider = *ride;
        rider.tiles = static_cast<unsigned>(tiles_m) * tiles_n;
        rider.front = rider.tiles >= 512;                       // several rounds of tiles: ride in the first one
        ride->blocks = 0;                                       // taken
    }
    const dim3 grid(static_cast<unsigned>(tiles_m) * tiles_n + rider.blocks, ny, bt.count), block(NT);
    const int group_m = 8;
#define FXP_GEMM_LAUNCH(MODE)                                                                                      \
    hipLaunchKernelGGL((k_gemm_nt_dma<BM, BN, BK, WM, WN, STAGES, MODE, SCHED>), grid, block, 0, s, A, lda, B, ldb, C, \
                       ldc,                                                                                        \
                       static_cast<int>(M), static_cast<int>(N), static_cast<int>(K), k_per_split, eA, bitsA, eB,   \
                       bitsB, tiles_m, tiles_n, group_m, split_stride, bt.a, bt.b, bt.c, ConvTaps(), amax, rider)
    if (mode == kStoreI32) FXP_GEMM_LAUNCH(kStoreI32);
    else if (mode == kStoreF32) FXP_GEMM_LAUNCH(kStoreF32);
    else FXP_GEMM_LAUNCH(kAtomicI32);
#undef FXP_GEMM_LAUNCH
    return launch_status();
}

__global__ __launch_bounds__(256) void k_splitk_reduce(ReduceRider r) { splitk_reduce_body<true, 256>(r, blockIdx.x, gridDim.x); }

// workgroups of a reduction with `lanes` lanes per 16-byte piece of the output: 256 threads each, at most 2048
static unsigned reduce_blocks(const ReduceRider& r, int lanes) {
    const int64_t pieces = static_cast<int64_t>(r.M) * r.N / 4;
    return static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(2048, (pieces * lanes + 255) / 256)));
}

int splitk_reduce_launch(ReduceRider r, hipStream_t s) {
    r.group = reduce_lanes(static_cast<int64_t>(r.M) * r.N / 4, r.splits);
    r.blocks = reduce_blocks(r, r.group);
    hipLaunchKernelGGL(k_splitk_reduce, dim3(r.blocks), dim3(256), 0, s, r);
    return launch_status();
}

// How a product is cut up.  Depends on the shape only, so that workspace sizing and launch agree.
struct GemmPlan {
    bool use256;   // 256 x 256 tiles, else 128 x 128
    int splits;    // slices of the contraction (grid.y)
    bool tall;     // split products only: 128 x 256 tiles (use256 is false then)
};

// no slice longer than one int32 sum can hold
static GemmPlan long_contraction(GemmPlan p, int64_t K) {
    if (K > kMaxContraction) p.splits = static_cast<int>(std::max<int64_t>(p.splits, (K + kMaxSlice - 1) / kMaxSlice));
    return p;
}

static GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K) {
    const int num_cu = 256;
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256);
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128);
    const bool wide = M >= 256 && N >= 256;
    GemmPlan p{wide && t256 >= 96, 1, false};
    if (K >= 2048 && t256 < 64) {
        // small output, long contraction (a weight gradient): fill the chip along K, slices of 1024 or more
        if (wide && t256 >= 16) {
            // 128 x 256 tiles, about one workgroup per CU: measured on the ViT weight gradients (contraction 12608)
            // 768 x 2304: 30.8 us (4 slices) against 31.9 with 256 x 256 tiles and 7 slices; 768 x 3072: 39.0 (3)
            // against 39.5 (7) - and fewer slices to write and to sum afterwards.  Smaller outputs (768 x 768) stay
            // with 128 x 128 tiles: 19.6 us with the sum of their 7 slices against 22.0 (12 slices).
            const int64_t tiles = ((M + 127) / 128) * ((N + 255) / 256);
            p.use256 = false;
            p.tall = true;
            p.splits = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(num_cu / tiles, K / 1024)));
            return long_contraction(p, K);
        }
        p.use256 = false;
        p.splits = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((num_cu + t128 / 2) / t128, K / 1024)));
    }
    return long_contraction(p, K);
}

// elements between two workspace slices of an M x N product: a multiple of 4, so that every slice starts 16-byte
// aligned and the reduction can read all of them in 16-byte pieces
static int64_t slice_stride(int64_t M, int64_t N) { return (M * N + 3) / 4 * 4; }

// Output elements the busiest CU computes with 256 x 256 tiles (one workgroup per CU) and with 160 x 128 tiles
// (tiles dealt round-robin, two resident per CU): the smaller tiles win when they cut that by a quarter or more,
// i.e. when the large tiles leave many CUs idle or a last round nearly empty.
static bool fits_160x128(int64_t M, int64_t N) {
    const int64_t num_cu = 256;
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256), t160 = ((M + 159) / 160) * ((N + 127) / 128);
    const int64_t work256 = (t256 + num_cu - 1) / num_cu * (256 * 256), work160 = (t160 + num_cu - 1) / num_cu * (160 * 128);
    return 4 * work160 <= 3 * work256;
}

size_t gemm_split_ws_bytes(int64_t M, int64_t N, int64_t K) {
    const GemmPlan p = plan_gemm(M, N, K);
    return p.splits > 1 ? round_up(static_cast<size_t>(p.splits) * slice_stride(M, N) * sizeof(int32_t), 256) : 0;
}

// Register-staged products with fewer than two 128 x 128 tiles per CU (count: slices or matrices) take 64 x 64 tiles:
// they are bound by the latency of a step, and four times the workgroups hide it (1379 x 768 x 1000 has 66 large
// tiles for 256 CUs, 264 small ones).
static bool small_tiles(int64_t M, int64_t N, int64_t count) {
    return ((M + 127) / 128) * ((N + 127) / 128) * count < 512;
}

static Product make_product(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, const int8_t* B, int64_t ldb, void* C,
                            int64_t ldc, const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, uint32_t* amax, int tile) {
    Product p;
    p.A = A; p.B = B; p.C = C;
    p.lda = lda; p.ldb = ldb; p.ldc = ldc;
    p.M = static_cast<int>(M); p.N = static_cast<int>(N); p.K = static_cast<int>(K);
    p.eA = eA; p.eB = eB; p.bitsA = bitsA; p.bitsB = bitsB;
    p.amax = amax;
    p.tiles_m = static_cast<int>((M + tile - 1) / tile);
    p.tiles_n = static_cast<int>((N + tile - 1) / tile);
    p.tiles = static_cast<unsigned>(p.tiles_m) * p.tiles_n;
    return p;
}

static int launch_direct(const Product& p0, const Product& p1, bool fp32_out, hipStream_t s, ReduceRider* ride = nullptr) {
    ReduceRider rider;
    if (ride != nullptr && ride->blocks != 0) {
        rider = *ride;
        rider.tiles = p0.tiles + p1.tiles;
        ride->blocks = 0;                                       // taken
    }
    const dim3 grid(p0.tiles + p1.tiles + rider.blocks), block(256);
    if (fp32_out) hipLaunchKernelGGL((k_gemm_nt_direct<kStoreF32>), grid, block, 0, s, p0, p1, rider);
    else hipLaunchKernelGGL((k_gemm_nt_direct<kStoreI32>), grid, block, 0, s, p0, p1, rider);
    return launch_status();
}

// Two independent products with fp32 outputs (the gradients of one layer, or of `batch` matrices each) in one launch, where
// neither fills the chip; kNotApplicable: one launch each.  Such launches wait for each other longer than they run (a launch
// behind a launch takes 4.5 us): the gradients of a 1379 x 768 x 1000 layer 13.7 + 8.7 -> 13.4 us, of 256 x 256 x 256 4.7 + 4.6 -> 4.9, the second pair of 96 x (197 x 64 x 197) 6.5 + 6.9 -> 7.9.
int gemm_nt_pair_launch(const GemmArgs& a, const GemmArgs& b, int64_t batch, hipStream_t s) {
    auto product = [](const GemmArgs& g, int tile) {
        Product p = make_product(g.M, g.N, g.K, g.A, g.lda, g.B, g.ldb, g.C, g.ldc, g.eA, g.bitsA, g.eB, g.bitsB, nullptr, tile);
        p.batch_a = g.strideA; p.batch_b = g.strideB; p.batch_c = g.strideC;
        return p;
    };
    if (batch == 1 && direct_fits(a.M, a.N, a.K) && direct_fits(b.M, b.N, b.K))
        return launch_direct(product(a, 32), product(b, 32), true, s);
    // Where one of them lies off the 16-byte grid the staged kernel is its own; products that the direct-to-LDS kernels would take
    // gain by the common launch while their large tiles, of which each CU would have one or none, are fewer than two per CU together
    // (layer steps, two launches / one: 1024^3 40.0 / 31.8, 1376 x 768 x 1000 47.9 / 36.7, 2032 x 768 x 768 51.4 / 37.7, 640 x 1024 x
    // 640 36.9 / 30.1, 1600^3 - 338 large tiles - 57.4 / 55.3, 2001 x 1600 x 1600 - 377 - 71.1 / 66.9, 2001 x 2032 x 3072 - 640 - 123.2 /
    // 124.1).  Not in batches, which fill the chip (60 x 250 x 250 81.2 / 82.8).
    bool aligned_one = false;
    auto staged = [&](const GemmArgs& g) {
        const bool vec = aligned(g.A, 16) && aligned(g.B, 16) && g.lda % 16 == 0 && g.ldb % 16 == 0 && g.K % 16 == 0 &&
                         (batch == 1 || (g.strideA % 16 == 0 && g.strideB % 16 == 0));
        if (vec && g.K >= 64) aligned_one = true;
        return g.K >= 16 && g.K <= kMaxContraction && small_tiles(g.M, g.N, batch) &&
               (batch > 1 || (plan_gemm(g.M, g.N, g.K).splits == 1 && !direct_fits(g.M, g.N, g.K)));
    };
    if (!staged(a) || !staged(b)) return kNotApplicable;
    auto large_tiles = [](const GemmArgs& g) { return ((g.M + 127) / 128) * ((g.N + 127) / 128); };
    if (aligned_one && (batch > 1 || large_tiles(a) + large_tiles(b) >= 512)) return kNotApplicable;
    const Product two = product(b, 64);
    Batch bt;
    bt.count = static_cast<unsigned>(batch);
    bt.a = a.strideA; bt.b = a.strideB; bt.c = a.strideC;
    return launch_cfg<64, 64, 128, 32, 32>(a.M, a.N, a.K, a.A, a.lda, a.B, a.ldb, a.C, a.ldc, kStoreF32, 1, a.eA, a.bitsA, a.eB,
                                           a.bitsB, s, 0, nullptr, bt, nullptr, nullptr, two);
}

// `batch` products of one shape in one launch (grid.z), never split along K.
int gemm_nt_batched_launch(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, int64_t strideA,
                           const int8_t* B, int64_t ldb, int64_t strideB, void* C, int64_t ldc, int64_t strideC,
                           int64_t batch, bool fp32_out, const int32_t* eA, int bitsA, const int32_t* eB, int bitsB,
                           hipStream_t s) {
    // the batch supplies the parallelism: no split along K, tiles chosen per matrix
    if (M == 0 || N == 0 || batch == 0) return FXP_OK;
    const bool vec = aligned(A, 16) && aligned(B, 16) && lda % 16 == 0 && ldb % 16 == 0 && K % 16 == 0 && strideA % 16 == 0 &&
                     strideB % 16 == 0;
    const bool dma = vec && K >= 64;   // K % 16 == 0: the direct-to-LDS kernels pad a partial last step with zeros
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256);
    const bool use256 = M >= 256 && N >= 256 && t256 * batch >= 96;
    const int mode = fp32_out ? kStoreF32 : kStoreI32;
    Batch bt;
    bt.count = static_cast<unsigned>(batch);
    bt.a = strideA; bt.b = strideB; bt.c = strideC;
#define FXP_BATCHED_ARGS M, N, K, A, lda, B, ldb, C, ldc, mode
#define FXP_BATCHED_TAIL 1, eA, bitsA, eB, bitsB, s, 0, nullptr, bt
    if (!dma) {
        // narrow outputs (head width 64 of the attention context and of dQ, dK, dV) take a tile of their own width
        if (small_tiles(M, N, batch)) return launch_cfg<64, 64, 128, 32, 32>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
        // matrices of one tile and one step (4096 x (32 x 32 x 32) attention step 137 us, in tiles of 128 rows 164)
        if (M <= 64 && N <= 64 && K <= 64) return launch_cfg<64, 64, 64, 32, 32>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
        if (N <= 64) return launch_cfg<128, 64, 64, 64, 32>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
        if (M <= 64) return launch_cfg<64, 128, 64, 32, 64>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
        return launch_cfg<128, 128, 64, 64, 64>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
    }
    if (use256 && K % 128 == 0) return launch_ring<64, 128>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
    if (use256) return launch_dma<256, 256, 64, 64, 128, 4>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
    // narrow outputs (head width 64 of the attention context and of dQ, dK, dV): a tile of their own width
    if (N <= 64) return launch_dma<128, 64, 64, 64, 32, 4>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
    // one or two steps along K (scores = Q K^T with head width 64): two stages, more workgroups per CU
    if (K <= 128) return launch_dma<128, 128, 64, 64, 64, 2>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
    if (K % 128 == 0) return launch_dma<128, 128, 128, 64, 32, 4>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
    return launch_dma<128, 128, 64, 64, 64, 4>(FXP_BATCHED_ARGS, FXP_BATCHED_TAIL);
#undef FXP_BATCHED_ARGS
#undef FXP_BATCHED_TAIL
}

// C = A[M,K] * B[N,K]^T.  fp32_out: C receives the inverse-mapped fp32 values (eA, eB on
// the device), else the int32 sums.  C is overwritten in both cases.
//
// Kernel choice (measured on MI355X with mapped Gaussian operands):
//   * small outputs of at most 1024 terms, whatever the alignment -> k_gemm_nt_direct (direct_fits);
//   * operands 16-byte aligned, K a multiple of 16 and 64 or more -> direct-to-LDS kernels, else the register-staged
//     kernel (k_gemm_nt: whole 16-byte loads at any byte address), 64 x 64 x 128 tiles below 512 large ones
//     (small_tiles), else 128 x 128 x 64;
//   * enough 256 x 256 tiles to fill the chip -> the ring kernel (K % 128 == 0) or the
//     four-stage 256 x 256 x 64 kernel; otherwise 128 x 128 tiles, or 64 x 64 (quarter_tiles);
//   * output-bound products (below the ridge, wide and large output or a very short contraction) -> 128-row tiles
//     of 64 or 96 KiB of LDS, so that two workgroups are resident per CU and one stores while the other multiplies;
//   * long contraction and a small output (the weight gradient) -> split K over grid.y.
//     With workspace every slice stores its own int32 matrix and one pass sums the slices
//     and applies the inverse mapping; without it the slices add into the zeroed output
//     with int32 atomics (device-scope atomics are served at the memory side on this
//     multi-die part, about 4x slower) and a pass converts in place.  Both are exact.
//
// amax (fp32_out only, may be null): FXP_ABSMAX_WORDS device words raised so that their maximum is at least the
// IEEE bits of the largest |C| of this product.
// ride (may be null): a pending reduction of another product; if this product is launched unsplit it takes the
// reduction along (ride->blocks becomes 0), otherwise the caller still has to launch it.
// defer (may be null): if this product is split along K into workspace slices, its reduction is not launched but
// described in *defer (blocks != 0) for the caller to send along with a later launch or to launch by itself;
// the slices in ws must stay untouched until then.
int gemm_nt_launch(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, const int8_t* B, int64_t ldb,
                   void* C, int64_t ldc, bool fp32_out, const int32_t* eA, int bitsA, const int32_t* eB, int bitsB,
                   void* ws, size_t ws_bytes, hipStream_t s, uint32_t* amax, ReduceRider* ride, ReduceRider* defer) {
    if (M == 0 || N == 0) return FXP_OK;
    if (!fp32_out) amax = nullptr;
    if (direct_fits(M, N, K))
        return launch_direct(make_product(M, N, K, A, lda, B, ldb, C, ldc, eA, bitsA, eB, bitsB, amax, 32), Product(), fp32_out, s, ride);
    uint32_t* amax1 = nullptr;      // the product kernel publishes the maximum itself only when it writes the final fp32
    const bool vec = aligned(A, 16) && aligned(B, 16) && lda % 16 == 0 && ldb % 16 == 0 && K % 16 == 0;
    const bool dma = vec && K >= 64;   // K % 16 == 0: the direct-to-LDS kernels pad a partial last step with zeros
    const GemmPlan plan = plan_gemm(M, N, K);
    const int splits = plan.splits;
    const bool use256 = plan.use256;
    // HBM-bound by the roofline (below 625 operations per byte) with the output stream dominating: a very short
    // contraction or an output of 128 MB and more (measured: c2 dX 26.6 -> 25.0 us, ViT fc1 forward 59 -> 53 us; the
    // 256 x 256 ring kernel stays ahead on the narrower and smaller outputs)
    const bool hbm_bound = 2.0 * M * N * K < 625.0 * (static_cast<double>(M) * K + static_cast<double>(N) * K + 4.0 * M * N);
    const bool stream_out = hbm_bound && N >= 1024 && (K <= 256 || 4.0 * M * N >= 96.0 * 1024 * 1024);
    const bool to_ws = splits > 1 && ws != nullptr && aligned(ws, 16) && ws_bytes >= gemm_split_ws_bytes(M, N, K);
    const int first_mode = splits > 1 ? (to_ws ? kStoreI32 : kAtomicI32) : (fp32_out ? kStoreF32 : kStoreI32);
    void* dst = to_ws ? ws : C;
    const int64_t dst_ld = to_ws ? N : ldc;
    const int64_t split_stride = to_ws ? slice_stride(M, N) : 0;
    // beyond kMaxContraction only the 64-bit sum of workspace slices is exact
    if (K > kMaxContraction && !(to_ws && fp32_out)) return FXP_ERR_OVERFLOW;
    int hr, hc;
    dim3 hgrid;
    rows_launch_shape(M, N, ldc, &hr, &hc, &hgrid);
    if (splits == 1) amax1 = amax;
    const Batch one{};
    int rc, slices = 1;   // the launchers round a slice up to whole K steps, so fewer slices than planned may run
    if (splits > 1 && !to_ws) {
        hipLaunchKernelGGL(k_zero_rows, hgrid, dim3(256), 0, s, static_cast<int32_t*>(C), ldc, hr, hc);
        if ((rc = launch_status())) return rc;
    }
    if (!dma && small_tiles(M, N, splits))
        rc = launch_cfg<64, 64, 128, 32, 32>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, splits, eA, bitsA, eB, bitsB, s, split_stride, &slices, one, amax1, ride);
    else if (!dma)
        rc = launch_cfg<128, 128, 64, 64, 64>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, splits, eA, bitsA, eB, bitsB, s, split_stride, &slices, one, amax1, ride);
    else if (use256 && splits == 1 && stream_out && K % 128 == 0 && (K <= 256 || 4.0 * M * N < 128.0 * 1024 * 1024))
        // 64 KiB of LDS per workgroup keeps two resident per CU: one stores its tile while the other multiplies
        // (ResNet dX 25088 x 1152 x 128: 22.5 us against 27.3 with the 128 x 256 tile and 24.4 with the ring kernel;
        // ViT qkv forward 36.7 / 38.3 / 40.5; fc1 forward 48.1 / 46.9 / 54.7)
        rc = launch_dma<128, 128, 128, 64, 64, 2>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, 1, eA, bitsA, eB, bitsB, s, 0, nullptr, one, amax1, ride);
    else if (use256 && splits == 1 && stream_out)
        rc = launch_dma<128, 256, 64, 64, 64, 3>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, 1, eA, bitsA, eB, bitsB, s, 0, nullptr, one, amax1, ride);
    else if (use256 && K % 128 == 0 && splits == 1 && fits_160x128(M, N))
        // too few 256 x 256 tiles for the 256 CUs: 160 x 128 tiles, two workgroups resident per CU (one is at its
        // barrier or in its epilogue while the other multiplies).  ViT-B, 12608 x 768 outputs = 150 tiles of 256 x 256
        // against 474 of these: contraction 3072: 39.9 -> 35.2 us, 2304: 32.4 -> 28.1, 768: 16.8 -> 14.7
        rc = launch_dma<160, 128, 128, 160, 32, 2>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, 1, eA, bitsA, eB, bitsB, s, 0, nullptr, one, amax1, ride);
    else if (use256 && K % 128 == 0 && splits == 1)
        rc = launch_ring<64, 128>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, 1, eA, bitsA, eB, bitsB, s, 0, nullptr, one, amax1, ride);
    else if (plan.tall)
        rc = launch_dma<128, 256, 64, 64, 64, 3>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, splits, eA, bitsA, eB, bitsB, s, split_stride, &slices, one, amax1, ride);
    else if (use256)
        rc = launch_dma<256, 256, 64, 64, 128, 4>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, splits, eA, bitsA, eB, bitsB, s, split_stride, &slices, one, amax1, ride);
    else if (splits == 1 && K % 128 == 0 && quarter_tiles(M, N, K, amax != nullptr))
        rc = launch_dma<64, 64, 128, 32, 32, 4>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, 1, eA, bitsA, eB, bitsB, s, 0, nullptr, one, amax1, ride);
    else if (splits == 1 && quarter_tiles(M, N, K, amax != nullptr))
        rc = launch_dma<64, 64, 64, 32, 32, 4>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, 1, eA, bitsA, eB, bitsB, s, 0, nullptr, one, amax1, ride);
    else if (K % 128 == 0)
        rc = launch_dma<128, 128, 128, 64, 32, 4>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, splits, eA, bitsA, eB, bitsB, s, split_stride, &slices, one, amax1, ride);
    else
        rc = launch_dma<128, 128, 64, 64, 64, 4>(M, N, K, A, lda, B, ldb, dst, dst_ld, first_mode, splits, eA, bitsA, eB, bitsB, s, split_stride, &slices, one, amax1, ride);
    if (rc || splits == 1) return rc;
    if (to_ws) {
        ReduceRider r;
        r.parts = static_cast<const int32_t*>(ws);
        r.splits = slices;
        r.stride = split_stride;
        r.M = static_cast<int>(M);
        r.N = static_cast<int>(N);
        r.C = C;
        r.ldc = ldc;
        r.fp32_out = fp32_out ? 1 : 0;
        r.eA = eA; r.bitsA = bitsA; r.eB = eB; r.bitsB = bitsB;
        r.amax = amax;
        r.wide = K > kMaxContraction ? 1 : 0;
        if (defer != nullptr) {
            r.blocks = reduce_blocks(r, 1);
            *defer = r;
            return FXP_OK;
        }
        return splitk_reduce_launch(r, s);
    }
    if (!fp32_out) return rc;
    hipLaunchKernelGGL(k_unmap_rows, hgrid, dim3(256), 0, s, static_cast<int32_t*>(C), ldc, hr, hc, eA, bitsA, eB, bitsB, amax);
    return launch_status();
}

// Y[M, Cout] = unmap(patches(Xq) * Wq^T) with the patch matrix never stored (see k_gemm_nt_dma, CONV): M output
// pixels, K = KH*KW*C.  Returns kNotApplicable when the shape needs the explicit patch matrix: channels not a
// multiple of 64 (the smallest K step), a long contraction in few tiles (deep_chain), or a 1x1 layer that plan_gemm gives
// 256 x 256 tiles.  For these neither way is ahead throughout (layer steps in us, with those tiles / here: 64 x 14 x 14 x 1024
// -> 1024 130.6 / 138.6, 64 x 28 x 28 x 128 -> 256 77.7 / 78.2, but 256 -> 512 141 / 135, 32 x 28 x 28 x 512 -> 256 90.7 / 84.2,
// 32 x 56 x 56 x 256 181 / 172); of a 3x3 layer the stored patches cost more than the larger tiles gain (64 x 14 x 14 x 256 ->
// 512 135 / 125).
template <int BM, int BN, int BK, int WM, int WN, int STAGES = 4>
static int conv_gemm_launch_cfg(const ConvTaps& ct, int64_t K, int64_t M, int64_t Cout, const int8_t* Xq, const int8_t* Wq,
                                float* Y, const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, hipStream_t s,
                                ReduceRider* ride) {
    const int tiles_m = static_cast<int>((M + BM - 1) / BM), tiles_n = static_cast<int>((Cout + BN - 1) / BN);
    ReduceRider rider;
    if (ride != nullptr && ride->blocks != 0) {
        rider = *ride;
        rider.tiles = static_cast<unsigned>(tiles_m) * tiles_n;
        rider.front = rider.tiles >= 512;                       // several rounds of tiles: ride in the first one
        ride->blocks = 0;                                       // taken
    }
    const dim3 grid(static_cast<unsigned>(tiles_m) * tiles_n + rider.blocks), block((BM / WM) * (BN / WN) * 64);
    hipLaunchKernelGGL((k_gemm_nt_dma<BM, BN, BK, WM, WN, STAGES, kStoreF32, true, true>), grid, block, 0, s, Xq, K, Wq, K,
                       static_cast<void*>(Y), Cout, static_cast<int>(M), static_cast<int>(Cout), static_cast<int>(K),
                       static_cast<int>(K), eA, bitsA, eB, bitsB, tiles_m, tiles_n, 8, int64_t{0}, int64_t{0}, int64_t{0},
                       int64_t{0}, ct, static_cast<uint32_t*>(nullptr), rider);
    return launch_status();
}

// Contractions that few tiles walk as one chain of steps for longer than it takes to store the patches and split the product.
// The chain grows with K, the stored patches with K and M.  Layer steps in us, stored and split / implicit: K = 9216, M = 16
// 122 / 142, 49 148 / 143, 98 151 / 146; 13824, 49 267 / 271, 98 272 / 277, 196 298 / 280; 18432, 98 377 / 382, 392 445 / 414,
// 784 104 / 106 (64 output channels); 36864, 128 240 / 275, 392 153 / 190 (64).  Of a 1x1 layer, whose patches are the image,
// K = 2048, M = 49 64.7 / 61.1, 4096, 49 143 / 154, 196 159 / 160.
static bool deep_chain(const ConvTaps& ct, int64_t M, int64_t K) {
    if (K == ct.C && ct.stride == 1 && ct.pad == 0 && ct.padw == 0) return K > 2048;
    return K > 4608 && (K > 18432 || K > 128 * M);
}

int conv_gemm_launch(const ConvTaps& ct, int KH, int64_t M, int64_t Cout, const int8_t* Xq, const int8_t* Wq, float* Y,
                     const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, hipStream_t s, ReduceRider* ride) {
    const int64_t K = static_cast<int64_t>(KH) * ct.KW * ct.C;
    if (ct.C % 64 != 0 || !aligned(Xq, 16) || !aligned(Wq, 16) || M <= 0 || Cout <= 0) return kNotApplicable;
    const GemmPlan plan = plan_gemm(M, Cout, K);
    if (plan.use256 && K == ct.C) return kNotApplicable;
    // few tiles: a product of stored patches would be split along K (or leave CUs idle); here tiles a quarter the size
    // fill more of the chip, no patches are stored and no slices summed.  Layer steps against stored patches: 32 x 14 x 14 x
    // 256 -> 256 3x3 110 -> 64 us (98 large tiles), 32 x 7 x 7 x 512 113 -> 80 (52).  The line, 64 x 64 / large tiles: 96
    // (37 x 14 x 14 x 512) 120 / 126, 92 (29 x 14 x 14 x 256) 86 / 90, 112 (36) 68.5 / 70.3, 130 (42) 117.5 / 103.7, 192 140.7 / 128.5.
    // (Of contractions up to 4608 every size down to one image of 4 x 4 gains: 1 x 7 x 7 x 512 95.6 -> 70.9, 1 x 4 x 4 x 256
    // 60.2 -> 45.1.)
    const int64_t t128 = ((M + 127) / 128) * ((Cout + 127) / 128);
    if (t128 <= 128) {
        if (plan.splits > 1 && deep_chain(ct, M, K)) return kNotApplicable;
        if (ct.C % 128 == 0) return conv_gemm_launch_cfg<64, 64, 128, 32, 32>(ct, K, M, Cout, Xq, Wq, Y, eA, bitsA, eB, bitsB, s, ride);
        return conv_gemm_launch_cfg<64, 64, 64, 32, 32>(ct, K, M, Cout, Xq, Wq, Y, eA, bitsA, eB, bitsB, s, ride);
    }
    // up to 64 output channels: a tile of their own width and three workgroups per CU (32 x 56 x 56 x 64 -> 64 3x3 layer step
    // 102.2 -> 88.7 us, 1x1 66.9 -> 61.8).
    // one K step = one run of channels of one filter tap: 128 channels (8 waves) where C allows, else 64 (4 waves)
    if (Cout <= 64) return conv_gemm_launch_cfg<128, 64, 64, 64, 32>(ct, K, M, Cout, Xq, Wq, Y, eA, bitsA, eB, bitsB, s, ride);
    // more tiles than CUs: two stages leave room for two workgroups per CU, one stores while the other multiplies, and the last
    // round is fuller (layer steps 64 x 28 x 28 x 128 3x3 100.7 -> 91.5 us, 64 x 28 x 28 x 256 -> 512 415 -> 370, 64 x 14 x 14 x 512
    // 192 -> 172; 128 x 64 tiles of two stages 101, 391, 210)
    if (ct.C % 128 == 0 && t128 > 256)
        return conv_gemm_launch_cfg<128, 128, 128, 64, 32, 2>(ct, K, M, Cout, Xq, Wq, Y, eA, bitsA, eB, bitsB, s, ride);
    if (ct.C % 128 == 0) return conv_gemm_launch_cfg<128, 128, 128, 64, 32>(ct, K, M, Cout, Xq, Wq, Y, eA, bitsA, eB, bitsB, s, ride);
    return conv_gemm_launch_cfg<128, 128, 64, 64, 64>(ct, K, M, Cout, Xq, Wq, Y, eA, bitsA, eB, bitsB, s, ride);
}

// dX[N, H, W, C] of a strided convolution from dYq[N, Ho, Wo, Cout] and the weights in class order (StrideClasses): the
// channels of the gradient must fill whole K steps.
//
// Against the stored patch gradient (which may be split along its contraction) the longest class must not be a long
// serial chain in few tiles.  Layer steps in us, patch gradient / classes, at contraction length (tiles): 512 (196) 69 / 53;
// 1024 (16) 50.1 / 48.7, (196) 87 / 67; 2048 (32) 56.8 / 59.8, (56) 57.4 / 59.8, (152) 84 / 72; 4096 (28) 78.7 / 83.5,
// (112) 80.2 / 87.6, (196) 103 / 94, (296) 126 / 121; 8192 (224) 169 / 180, (608) 315 / 339; 9216 (32) 68 / 105.
bool conv_strided_dx_fits(const StrideClasses& sc, int64_t images, int64_t C) {
    if (sc.stride <= 1 || sc.stride > kMaxStride || sc.C % 64 != 0) return false;
    int64_t row_tiles = 0, tiles = 0, longest = 0;
    for (int c = 0; c < sc.stride * sc.stride; ++c) {
        const StrideClass& k = sc.cls[c];
        const int64_t t = (images * k.Ho * k.Wo + 127) / 128;
        row_tiles = std::max(row_tiles, t * sc.stride * sc.stride);
        tiles += t * ((C + 127) / 128);
        longest = std::max(longest, static_cast<int64_t>(k.TH) * k.TW * sc.C);
    }
    return row_tiles < (int64_t{1} << 24) && (longest <= 1024 || (longest <= 4096 && longest <= 32 * tiles));
}

template <int BN, int BK, int WN, int STAGES = 4>
static int conv_strided_dx_cfg(const StrideClasses& sc, int64_t images, int64_t C, const int8_t* dYq, const int8_t* Wc, float* dX,
                               const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, hipStream_t s, ReduceRider* ride) {
    constexpr int BM = 128, WM = 64;
    int64_t rows = 0;
    for (int c = 0; c < sc.stride * sc.stride; ++c) rows = std::max(rows, images * sc.cls[c].Ho * sc.cls[c].Wo);
    const int tiles_m = static_cast<int>((rows + BM - 1) / BM) * sc.stride * sc.stride, tiles_n = static_cast<int>((C + BN - 1) / BN);
    ReduceRider rider;
    if (ride != nullptr && ride->blocks != 0) {
        rider = *ride;
        rider.tiles = static_cast<unsigned>(tiles_m) * tiles_n;
        rider.front = rider.tiles >= 512;                       // several rounds of tiles: ride in the first one
        ride->blocks = 0;                                       // taken
    }
    const dim3 grid(static_cast<unsigned>(tiles_m) * tiles_n + rider.blocks), block((BM / WM) * (BN / WN) * 64);
    hipLaunchKernelGGL((k_gemm_nt_dma<BM, BN, BK, WM, WN, STAGES, kStoreF32, true, true, StrideClasses>), grid, block, 0, s, dYq,
                       int64_t{0}, Wc, int64_t{0}, static_cast<void*>(dX), C, static_cast<int>(images), static_cast<int>(C), 0, 0, eA,
                       bitsA, eB, bitsB, tiles_m, tiles_n, 8, int64_t{0}, int64_t{0}, int64_t{0}, int64_t{0}, sc,
                       static_cast<uint32_t*>(nullptr), rider);
    return launch_status();
}

int conv_strided_dx_launch(const StrideClasses& sc, int64_t images, int64_t C, const int8_t* dYq, const int8_t* Wc, float* dX,
                           const int32_t* eA, int bitsA, const int32_t* eB, int bitsB, hipStream_t s, ReduceRider* ride) {
    // as in conv_gemm_launch (48 x 56 x 56 x 64 -> 128 3x3 layer step 100.6 -> 83.6 us, 1x1 80.7 -> 66.5)
    if (C <= 64) return conv_strided_dx_cfg<64, 64, 32>(sc, images, C, dYq, Wc, dX, eA, bitsA, eB, bitsB, s, ride);
    int64_t tiles = 0;
    for (int c = 0; c < sc.stride * sc.stride; ++c) tiles += (images * sc.cls[c].Ho * sc.cls[c].Wo + 127) / 128 * ((C + 127) / 128);
    if (sc.C % 128 == 0 && tiles > 256) return conv_strided_dx_cfg<128, 128, 32, 2>(sc, images, C, dYq, Wc, dX, eA, bitsA, eB, bitsB, s, ride);
    if (sc.C % 128 == 0) return conv_strided_dx_cfg<128, 128, 32>(sc, images, C, dYq, Wc, dX, eA, bitsA, eB, bitsB, s, ride);
    return conv_strided_dx_cfg<128, 64, 64>(sc, images, C, dYq, Wc, dX, eA, bitsA, eB, bitsB, s, ride);
}

// long_k: the caller can take a contraction beyond kMaxContraction (fp32 output through workspace slices)
static int check_gemm_args(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, int transA, const void* B,
                           int64_t ldb, int transB, const void* C, int64_t ldc, bool long_k = false) {
    if (M < 0 || N < 0 || K < 0) return FXP_ERR_DIMS;
    if (M >= (int64_t{1} << 31) || N >= (int64_t{1} << 31) || K >= (int64_t{1} << 31)) return FXP_ERR_DIMS;
    if (K > kMaxContraction && !long_k) return FXP_ERR_OVERFLOW;
    if (lda < (transA ? M : K) || ldb < (transB ? K : N) || ldc < N) return FXP_ERR_DIMS;
    if ((M * N > 0 && !C) || (M * K > 0 && !A) || (N * K > 0 && !B)) return FXP_ERR_NULL;
    if (!aligned(C, 4)) return FXP_ERR_ALIGN;
    if (((M + 127) / 128) * ((N + 127) / 128) >= (int64_t{1} << 31)) return FXP_ERR_DIMS;
    return FXP_OK;
}

static size_t gemm_ws_bytes(int transA, int transB, int64_t M, int64_t N, int64_t K) {
    size_t b = 0;
    if (transA) b += round_up(static_cast<size_t>(M) * static_cast<size_t>(K), 256);
    if (!transB) b += round_up(static_cast<size_t>(N) * static_cast<size_t>(K), 256);
    return b;
}

size_t gemm_ws_worst(int64_t M, int64_t N, int64_t K) { return gemm_ws_bytes(1, 0, M, N, K) + gemm_split_ws_bytes(M, N, K); }

// Bring any operand form to the native one (transposed copies in ws), then run it.
static int gemm_any(int transA, int transB, int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda,
                    const int8_t* B, int64_t ldb, void* C, int64_t ldc, bool fp32_out, const int32_t* eA, int bitsA,
                    const int32_t* eB, int bitsB, void* ws, size_t ws_bytes, hipStream_t s, uint32_t* amax = nullptr) {
    if (M == 0 || N == 0) return FXP_OK;
    const size_t need = gemm_ws_bytes(transA, transB, M, N, K);
    if (need > 0 && (!ws || ws_bytes < need)) return FXP_ERR_WORKSPACE;
    if (ws && !aligned(ws, 256)) return FXP_ERR_ALIGN;
    // a contraction beyond one int32 sum needs the slice area behind the transposed copies (nothing is enqueued otherwise)
    if (K > kMaxContraction && (!fp32_out || !ws || ws_bytes < need + gemm_split_ws_bytes(M, N, K))) return FXP_ERR_OVERFLOW;
    int8_t* w = static_cast<int8_t*>(ws);
    int rc;
    if (transA && K > 0) {
        if ((rc = transpose_i8_launch(A, K, M, lda, w, s))) return rc;      // stored [K, M] -> [M, K]
        A = w;
        lda = K;
        w += round_up(static_cast<size_t>(M) * static_cast<size_t>(K), 256);
    }
    if (!transB && K > 0) {
        if ((rc = transpose_i8_launch(B, K, N, ldb, w, s))) return rc;      // stored [K, N] -> [N, K]
        B = w;
        ldb = K;
        w += round_up(static_cast<size_t>(N) * static_cast<size_t>(K), 256);
    }
    // what is left of the workspace serves the split-K slices (atomics are used if it is too small)
    const size_t used = static_cast<size_t>(w - static_cast<int8_t*>(ws));
    return gemm_nt_launch(M, N, K, A, lda, B, ldb, C, ldc, fp32_out, eA, bitsA, eB, bitsB, ws ? w : nullptr,
                          ws_bytes > used ? ws_bytes - used : 0, s, amax, nullptr, nullptr);
}

}  // namespace fxp

extern "C" int fxp_gemm(int transA, int transB, int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda,
                        const int8_t* B, int64_t ldb, int32_t* C, int64_t ldc, void* ws, size_t ws_bytes, void* stream) {
    int rc = fxp::check_gemm_args(M, N, K, A, lda, transA, B, ldb, transB, C, ldc);
    if (rc) return rc;
    return fxp::gemm_any(transA, transB, M, N, K, A, lda, B, ldb, C, ldc, false, nullptr, 8, nullptr, 8, ws, ws_bytes,
                         static_cast<hipStream_t>(stream));
}

extern "C" int fxp_gemm_unmap(int transA, int transB, int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda,
                              const int8_t* B, int64_t ldb, const int32_t* eA, int bitsA, const int32_t* eB, int bitsB,
                              float* C, int64_t ldc, void* ws, size_t ws_bytes, void* stream) {
    int rc = fxp::check_gemm_args(M, N, K, A, lda, transA, B, ldb, transB, C, ldc, true);
    if (rc) return rc;
    if (!eA) return FXP_ERR_NULL;
    if (bitsA < 2 || bitsA > 8 || (eB && (bitsB < 2 || bitsB > 8))) return FXP_ERR_BITS;
    return fxp::gemm_any(transA, transB, M, N, K, A, lda, B, ldb, C, ldc, true, eA, bitsA, eB, bitsB, ws, ws_bytes,
                         static_cast<hipStream_t>(stream));
}

extern "C" int fxp_gemm_unmap_absmax(int transA, int transB, int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda,
                                     const int8_t* B, int64_t ldb, const int32_t* eA, int bitsA, const int32_t* eB,
                                     int bitsB, float* C, int64_t ldc, uint32_t* out_absmax, void* ws, size_t ws_bytes,
                                     void* stream) {
    int rc = fxp::check_gemm_args(M, N, K, A, lda, transA, B, ldb, transB, C, ldc, true);
    if (rc) return rc;
    if (!eA || !out_absmax) return FXP_ERR_NULL;
    if (!fxp::aligned(out_absmax, 4)) return FXP_ERR_ALIGN;
    if (bitsA < 2 || bitsA > 8 || (eB && (bitsB < 2 || bitsB > 8))) return FXP_ERR_BITS;
    return fxp::gemm_any(transA, transB, M, N, K, A, lda, B, ldb, C, ldc, true, eA, bitsA, eB, bitsB, ws, ws_bytes,
                         static_cast<hipStream_t>(stream), out_absmax);
}

// Batched products for the attention matmuls (Q K^T and P V with per-tensor scales): `batch` independent
// C_b[M,N] = A_b[M,K] * B_b[N,K]^T, matrices of one operand strideX elements apart.
static int check_batched(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, int64_t strideA, const void* B,
                         int64_t ldb, int64_t strideB, const void* C, int64_t ldc, int64_t strideC, int64_t batch) {
    if (batch < 0 || batch > 65535 || strideA < 0 || strideB < 0 || strideC < 0) return FXP_ERR_DIMS;
    int rc = fxp::check_gemm_args(M, N, K, A, lda, 0, B, ldb, 1, C, ldc);
    if (rc) return rc;
    if (batch > 1 && M * N > 0 && strideC < (M - 1) * ldc + N) return FXP_ERR_DIMS;   // outputs must not overlap
    return FXP_OK;
}

extern "C" int fxp_gemm_batched(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, int64_t strideA,
                                const int8_t* B, int64_t ldb, int64_t strideB, int32_t* C, int64_t ldc, int64_t strideC,
                                int64_t batch, void* stream) {
    int rc = check_batched(M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch);
    if (rc) return rc;
    return fxp::gemm_nt_batched_launch(M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch, false, nullptr, 8,
                                       nullptr, 8, static_cast<hipStream_t>(stream));
}

extern "C" int fxp_gemm_unmap_batched(int64_t M, int64_t N, int64_t K, const int8_t* A, int64_t lda, int64_t strideA,
                                      const int8_t* B, int64_t ldb, int64_t strideB, const int32_t* eA, int bitsA,
                                      const int32_t* eB, int bitsB, float* C, int64_t ldc, int64_t strideC, int64_t batch,
                                      void* stream) {
    int rc = check_batched(M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch);
    if (rc) return rc;
    if (!eA) return FXP_ERR_NULL;
    if (bitsA < 2 || bitsA > 8 || (eB && (bitsB < 2 || bitsB > 8))) return FXP_ERR_BITS;
    return fxp::gemm_nt_batched_launch(M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch, true, eA, bitsA, eB,
                                       bitsB, static_cast<hipStream_t>(stream));
}
