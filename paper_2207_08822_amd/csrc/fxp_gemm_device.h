// Device code that the product kernels share: operand and accumulator types, LDS swizzle, waits, the epilogue.
#pragma once
#include "fxp_internal.h"

namespace fxp {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

enum { kStoreI32 = 0, kStoreF32 = 1, kAtomicI32 = 2 };

template <int V>
using IC = std::integral_constant<int, V>;

constexpr int kNumXcd = 8;

template <int BK>
__device__ inline int swizzle_of_row(int row) {
    constexpr int CPR = BK / 16;            // 16-byte pieces per LDS row
    return (row / (16 / CPR)) % CPR;        // period 16 rows: 16 rows x 16 B = all 64 banks once
}

// The wave's largest output magnitude -> one of the FXP_ABSMAX_WORDS words at amax (IEEE bits of a non-negative
// float order like unsigned integers): one device-scope atomic per wave, without a returned value and with no
// load before it - vector memory operations complete in order, so anything a wave has to WAIT for behind its
// stores (a look at the word first, to skip the atomic) keeps it alive until they have drained, and the
// output-bound products live on waves ending while their stores are still in flight; consecutive waves use
// words in different cache lines, those of a workgroup of four (64 x 64 tiles, the most of them) and of the next one all eight: with
// four lines for all workgroups of four 8000 x 256 x 384 took 9.6 us, 7.3 so; 256 x 7232 x 768 10.0 / 7.9.
__device__ inline void publish_absmax(float m, uint32_t* amax) {
    const uint32_t b = wave_max(__float_as_uint(m));
    // (block and thread indices only: the launch dimensions would be LOADED, and a wave that waits for a load
    // behind its stores stays alive until they have drained)
    const unsigned group = blockIdx.x + blockIdx.y * 37u, line = (4 * group + (threadIdx.x >> 6)) & 7u, word = (group >> 1) & 31u;
    if ((threadIdx.x & 63) == 0) atomicMax(amax + (line * 32u + word), b);     // 8 lines of 32 words
}

// Epilogue of every product kernel: the wave's FM x FN fragments of 32 x 32 go to C (top-left element row0, col0
// of the wave's tile), as inverse-mapped fp32 (non-temporal: the output is not read again here), as int32, or
// added into int32 with atomics.  Accumulator register r of lane l is row 8 * (r / 4) + 4 * (l / 32) + r % 4,
// column l % 32 of its fragment.  AMAX: returns the largest magnitude this lane stored.
// GUARD = false: the wave's tile lies inside C - no bounds tests, row addresses a scalar multiple of ldc away from
// the lane's base.  PLAIN: 2^E is a normal float (or the output is int32) - one convert and one multiply per
// value.  The output-bound products spend a fifth of their time issuing this loop, so both tests are made once
// per wave, outside it.
template <int FM, int FN, int MODE, bool AMAX, bool GUARD, bool PLAIN>
__device__ inline float store_loop(const v16i (&acc)[FM][FN], void* __restrict__ Cv, int64_t ldc, int M, int N, int row0,
                                   int col0, int fhalf, int frow, int E) {
    float m = 0.0f;
    const float unit = __uint_as_float(static_cast<uint32_t>(PLAIN ? E + 127 : 127) << 23);
    const int64_t base = static_cast<int64_t>(row0 + 4 * fhalf) * ldc + col0 + frow;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int dr = 32 * i + 8 * (r >> 2) + (r & 3);            // row of this register below the lane's base row
            if (GUARD && row0 + 4 * fhalf + dr >= M) continue;
            const int64_t off_row = base + dr * ldc;
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (GUARD && col0 + 32 * j + frow >= N) continue;
                const int64_t off = off_row + 32 * j;
                if (MODE == kStoreF32) {
                    const float v = PLAIN ? static_cast<float>(acc[i][j][r]) * unit : unmap_value(acc[i][j][r], E);
                    __builtin_nontemporal_store(v, static_cast<float*>(Cv) + off);
                    if (AMAX) m = fmaxf(m, fabsf(v));
                } else if (MODE == kStoreI32) {
                    static_cast<int32_t*>(Cv)[off] = acc[i][j][r];
                } else {
                    atomicAdd(static_cast<int32_t*>(Cv) + off, acc[i][j][r]);
                }
            }
        }
    }
    return m;
}

template <int FM, int FN, int MODE, bool AMAX>
__device__ inline float store_fragments(const v16i (&acc)[FM][FN], void* __restrict__ Cv, int64_t ldc, int M, int N, int row0,
                                        int col0, int fhalf, int frow, int E) {
    const bool inside = row0 + 32 * FM <= M && col0 + 32 * FN <= N;                     // wave-uniform
    const bool plain = MODE != kStoreF32 || (E >= -126 && E <= 127);
    if (inside && plain) {
        float m = 0.0f;
        if (AMAX) {
            // the inverse mapping is monotone: the largest magnitude comes from the largest or the smallest sum,
            // found on the integers (one three-input max / min per value) before the store loop starts
            int hi = 0, lo = 0;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        hi = max(max(hi, acc[i][j][r]), acc[i][j][r + 1]);
                        lo = min(min(lo, acc[i][j][r]), acc[i][j][r + 1]);
                    }
            const float unit = __uint_as_float(static_cast<uint32_t>(E + 127) << 23);
            m = fmaxf(static_cast<float>(hi) * unit, -(static_cast<float>(lo) * unit));
        }
        store_loop<FM, FN, MODE, false, false, true>(acc, Cv, ldc, M, N, row0, col0, fhalf, frow, E);
        return m;
    }
    if (plain) return store_loop<FM, FN, MODE, AMAX, true, true>(acc, Cv, ldc, M, N, row0, col0, fhalf, frow, E);
    return store_loop<FM, FN, MODE, AMAX, true, false>(acc, Cv, ldc, M, N, row0, col0, fhalf, frow, E);
}

// s_waitcnt immediate (gfx9 encoding): wait until at most `vm` vector-memory operations
// and no LDS operation of this wave are outstanding.
__host__ __device__ constexpr int waitcnt_vm_lgkm0(int vm) { return (vm & 0xF) | ((vm >> 4) << 14) | 0x70; }

template <int VM>
__device__ inline void wait_loads_and_lds() {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(VM));
}

// 256 zero bytes: where the patch rows of an implicit convolution read their padding from, and a partial last K step
// the pieces beyond the end of the contraction
static __device__ __attribute__((aligned(256))) const uint8_t g_zero_page[256] = {0};

}  // namespace fxp
