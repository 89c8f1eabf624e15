// Device code that the mapping kernels share: the rounding of one element and of a quad of four (paper Sec. 3.1, App. A.1) and
// the scale a workgroup maps with.
#pragma once
#include "fxp_internal.h"

namespace fxp {

constexpr int kMapThreads = 256;

// 16 bytes at 4-byte alignment, 16 and 4 bytes at any alignment
struct __attribute__((packed, aligned(4))) Quad {
    uint32_t x, y, z, w;
};
struct __attribute__((packed, aligned(1))) Bytes16 {
    uint32_t x, y, z, w;
};
struct __attribute__((packed, aligned(1))) Bytes4 {
    uint32_t x;
};
__device__ inline uint4 load_quad(const uint32_t* p) {
    const Quad v = *reinterpret_cast<const Quad*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

struct MapCfg {
    int e_max;
    int cut;        // low bits dropped: 24 - (bits - 1)
    int rshift;     // 32 - cut: the random number is the top `cut` bits of the word
    uint32_t sat;   // 2^(bits-1) - 1
    uint32_t half;  // 2^(cut-1), the nearest-rounding increment
    uint32_t low_mask;  // 2^cut - 1
    float to_units;     // 2^(150 - e_max): |x| * to_units = the 24-bit mantissa shifted to the scale (e_max in [25, 254])
    float limit;        // 2^(e_max - 126): magnitudes from here on are above the scale (+Inf for e_max = 254)
};

// Magnitude of one element, every case: non-finite input, scale below the element.
template <bool STOCH>
__device__ inline uint32_t magnitude_full(uint32_t b, uint32_t word, const MapCfg& c) {
    const uint32_t e = (b >> 23) & 0xffu, f = b & 0x7fffffu;
    if (e == 255u) return f == 0u ? c.sat : 0u;
    const int d = c.e_max - static_cast<int>(max(e, 1u));
    if (d < 0) return c.sat;
    const uint32_t m = f | (e ? 0x800000u : 0u);
    const uint32_t mp = m >> min(d, 31);
    const uint32_t add = STOCH ? ((~word) >> c.rshift) : c.half;
    return min((mp + add) >> c.cut, c.sat);
}

// Same for the common case: e_max in [25, 254], no element above the scale, no result above the largest
// magnitude.  The shifted mantissa m >> (e_max - e) is the integer part of |x| * 2^(150 - e_max): the factor is a
// power of two (a normal float for these scales), so the product is exact whenever it is 1 or more and below 1
// otherwise, sub-normal inputs included, and the conversion truncates - two instructions for unpack, hidden
// bit, clamp and shift.  r < low  <=>  low + (2^cut - 1 - r) carries out of the cut.  `bad` collects, as a lane
// mask (one compare per element, accumulated on the scalar side), the lanes with an element the scale does not
// cover (exponent above it, Inf, NaN); the caller also ORs the results (a bit above the magnitude bits = needs
// the saturating path) and redoes the block with magnitude_full if either fires.
template <bool STOCH>
__device__ inline uint32_t magnitude_fast(uint32_t b, uint32_t word, const MapCfg& c, uint64_t& bad) {
    const float ax = fabsf(__uint_as_float(b));
    bad |= __builtin_amdgcn_ballot_w64(!(ax < c.limit));
    const uint32_t mp = static_cast<uint32_t>(ax * c.to_units);
    const uint32_t add = STOCH ? ((word >> c.rshift) ^ c.low_mask) : c.half;
    return (mp + add) >> c.cut;
}

__device__ inline uint32_t with_sign(uint32_t mag, uint32_t b) {
    const uint32_t sm = static_cast<uint32_t>(static_cast<int32_t>(b) >> 31);
    return (mag ^ sm) - sm;
}

// the four signed results of a 16-byte load as one dword, low bytes in element order
__device__ inline uint32_t pack4(uint32_t q0, uint32_t q1, uint32_t q2, uint32_t q3, const uint4 v) {
    const uint32_t p01 = perm(with_sign(q1, v.y), with_sign(q0, v.x), 0x0c0c0400u);
    const uint32_t p23 = perm(with_sign(q3, v.w), with_sign(q2, v.z), 0x0c0c0400u);
    return perm(p23, p01, 0x05040100u);
}


// the four mapped bytes of a quad: fast form (q_or and bad as above) and complete form
template <bool STOCH>
__device__ inline uint32_t map_quad_fast(const uint4 v, const uint4 w, const MapCfg& c, uint32_t& q_or, uint64_t& bad) {
    const uint32_t m0 = magnitude_fast<STOCH>(v.x, w.x, c, bad), m1 = magnitude_fast<STOCH>(v.y, w.y, c, bad);
    const uint32_t m2 = magnitude_fast<STOCH>(v.z, w.z, c, bad), m3 = magnitude_fast<STOCH>(v.w, w.w, c, bad);
    q_or |= m0 | m1 | m2 | m3;
    return pack4(m0, m1, m2, m3, v);
}

template <bool STOCH>
__device__ inline uint32_t map_quad_full(const uint4 v, const uint4 w, const MapCfg& c) {
    return pack4(magnitude_full<STOCH>(v.x, w.x, c), magnitude_full<STOCH>(v.y, w.y, c), magnitude_full<STOCH>(v.z, w.z, c),
                 magnitude_full<STOCH>(v.w, w.w, c), v);
}

__device__ inline MapCfg make_cfg(int e_max, int bits) {
    MapCfg c;
    c.e_max = e_max;
    c.cut = 24 - (bits - 1);
    c.rshift = 32 - c.cut;
    c.sat = (1u << (bits - 1)) - 1u;
    c.half = 1u << (c.cut - 1);
    c.low_mask = (1u << c.cut) - 1u;
    const int e = min(max(e_max, 25), 254);                       // outside: the fast path is not taken
    c.to_units = __uint_as_float(static_cast<uint32_t>(277 - e) << 23);
    c.limit = __uint_as_float(static_cast<uint32_t>(e + 1) << 23);
    return c;
}

// What this thread sees of the block maxima: loaded before the elements, so that their reduction can run while those are in flight (in
// k_map_tile; tiles of quads wait for both).
__device__ inline uint32_t partials_share(const uint32_t* partials, int n_partials) {
    if (partials == nullptr) return 0u;
    uint32_t m = static_cast<int>(threadIdx.x) < n_partials ? partials[threadIdx.x] : 0u;
    for (int i = threadIdx.x + kMapThreads; i < n_partials; i += kMapThreads) m = max(m, partials[i]);
    return m;
}

// scale of the tensor: either given, or the max of the per-block maxima (m: partials_share), and then published by one block
__device__ inline int resolve_scale(const int32_t* e_in, const uint32_t* partials, uint32_t m, int32_t* e_out, uint32_t* red,
                                    bool publish) {
    if (partials == nullptr) return e_in[0];
    m = block_max(m, red);
    const int e = max(1, static_cast<int>(m >> 23));
    if (publish && threadIdx.x == 0) e_out[0] = e;
    return e;
}

// A tensor wanted row-major only: quads of consecutive elements, 1024 * PASSES per workgroup from quad `first` on,
// whatever its rows are and wherever x and q start.  SHORT: the workgroup has fewer quads, and a last one that may be
// short; the others carry no bounds code (with it around every load, 12608 x 768 took 13.2 us where tiles take 10.6).
template <bool STOCH, int PASSES, bool SHORT, class Job>
__device__ inline void map_flat_body(const Job& J, int bits, bool publish, uint32_t* red, uint32_t key0, uint32_t key1,
                                     uint64_t first) {
    const uint64_t n = static_cast<uint64_t>(J.rows) * static_cast<uint64_t>(J.cols);
    const uint32_t quads = SHORT ? static_cast<uint32_t>((n >> 2) - first) : 4 * kMapThreads * PASSES;    // whole ones here
    const uint32_t tail = static_cast<uint32_t>(n & 3u);         // SHORT: elements of the quad behind them
    const uint32_t* __restrict__ x = J.x + 4 * first;
    int8_t* __restrict__ q = J.q + 4 * first;
    auto load_pass = [&](int p, uint4 (&v)[4]) {
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t i = (4 * p + k) * kMapThreads + threadIdx.x;
            if (!SHORT || i < quads) {
                v[k] = load_quad(x + 4 * i);
            } else {
                v[k] = make_uint4(0, 0, 0, 0);
                if (i == quads) {
                    if (tail > 0) v[k].x = x[4 * i];
                    if (tail > 1) v[k].y = x[4 * i + 1];
                    if (tail > 2) v[k].z = x[4 * i + 2];
                }
            }
        }
    };
    uint4 cur[4], nxt[4];
    const uint32_t share = partials_share(J.partials, J.n_partials);
    load_pass(0, cur);
    const MapCfg cfg = make_cfg(resolve_scale(J.e_in, J.partials, share, J.e_out, red, publish), bits);
    const bool scale_ok = cfg.e_max >= 25 && cfg.e_max < 255;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        if (p + 1 < PASSES) load_pass(p + 1, nxt);
        uint32_t o[4], q_or = 0;
        uint64_t bad = 0;
        auto words_of = [&](uint32_t k) {
            const uint64_t blk = first + ((4 * p + k) * kMapThreads + threadIdx.x);
            return STOCH ? philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(blk >> 32), J.sid0, J.sid1, key0, key1)
                         : make_uint4(0, 0, 0, 0);
        };
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) o[k] = map_quad_fast<STOCH>(cur[k], words_of(k), cfg, q_or, bad);
        if (!scale_ok || bad != 0 || (q_or & ~cfg.sat)) {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) o[k] = map_quad_full<STOCH>(cur[k], words_of(k), cfg);
        }
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t i = (4 * p + k) * kMapThreads + threadIdx.x;
            if (!SHORT || i < quads) {
                reinterpret_cast<Bytes4*>(q + 4 * i)->x = o[k];
            } else if (i == quads) {
                for (uint32_t j = 0; j < tail; ++j) q[4 * i + j] = static_cast<int8_t>(o[k] >> (8 * j));
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) cur[k] = nxt[k];
    }
}

}  // namespace fxp
