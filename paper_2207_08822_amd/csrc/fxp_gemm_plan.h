// How products are cut into slices and sums of slices among lanes: host arithmetic only, so that it can be checked without a device.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace fxp {

constexpr int64_t kMaxContraction = 133144;   // 127^2 * K < 2^31: the longest contraction one int32 sum can hold
// Longer contractions (a weight gradient over more rows than that) run as slices of at most kMaxSlice terms (a
// multiple of every K step), each summed exactly in int32 into its workspace slice; the slices are added in 64
// bits and the inverse mapping rounds that sum once.
constexpr int64_t kMaxSlice = 133120;

// Lanes of a wave that share a 16-byte piece of the output in a sum of slices that is a launch of its own.  One while the pieces alone
// fill the chip or the slices are few; else up to 32, each with eight slices - one round of loads - or more (a 64 x 147 output of 126
// slices: ten workgroups walked all slices in turn, 123 us; 256 slices with sixteen lanes 8.7 us, with 32 lanes 6.3; with four slices
// a lane the product and its sum take longer: 64 x 64 of 8 slices 9.3 -> 10.3 us, 256 x 256 of 8 10.0 -> 11.5, 512 x 512 of 12
// 16.9 -> 17.8, 64 x 64 of 128 11.3 -> 11.6).
inline int reduce_lanes(int64_t pieces, int64_t splits) {
    int lanes = 1;
    while (lanes < 32 && splits >= 16 * lanes && pieces * lanes < 65536) lanes *= 2;
    return lanes;
}

// Unsplit direct-to-LDS products of at most 128 large tiles, whatever they are for: half the CUs or more would have none, so tiles a
// quarter the size (the product alone, 128 x 128 / 64 x 64 tiles in us: 1024^3 7.3 / 5.5, M x N x K 512 x 3072 x 768 - 96 tiles - 7.6 /
// 6.6, 300 x 1000 x 2000 15.2 / 8.1, 16384 x 16 x 3072 14.9 / 10.9; also where large tiles would be padded by
// small ones, 1300 x 1400 x 2000 12.8 / 11.5).  Close to two small tiles a CU
// the gain is small, and it is lost where every row starts off the 64-byte grid and the contraction is long (480 and 512 small tiles:
// 1024 x 1920 x 2000 11.5 / 11.8, 1024 x 2048 x 2000 11.6 / 12.0, x 1520 9.6 / 9.9 but 1000 x 2000 x 1520 10.0 / 9.6; 448 small tiles
// 1024 x 1792 x 2000 11.4 / 11.2; at most 128 rows, whose operand all CUs share, 128 x 16384 x 2000 16.4 / 14.9), and in whole steps
// of 128 along a very long one (128 x 16384 x 4096 17.7 / 17.5, x 5120 21.7 / 22.7, x 8192 31.0 / 32.4, x 12288 43.6 / 46.7).
// Products that publish their largest magnitude do so once a wave, four times as often with small tiles: where many of them come to an
// end within a short contraction large ones are ahead (that product, large / small in us: 14848 x 128 x 128 6.2 / 6.6, 8000 x 256 x 128
// 6.3 / 6.8, 256 x 7232 x 256 6.5 / 6.8, 14976 x 128 x 448 7.0 / 7.1; 284 small tiles 9088 x 128 x 256 6.1 / 5.9, 452 of 256 x 7232 x 768
// 8.4 / 7.9).
inline bool quarter_tiles(int64_t M, int64_t N, int64_t K, bool absmax) {
    const int64_t large = ((M + 127) / 128) * ((N + 127) / 128), small = ((M + 63) / 64) * ((N + 63) / 64);
    if (large > 128 || (absmax && small > 340 && K <= 448)) return false;
    if (small <= 448 || small < 4 * large) return true;
    return K % 128 == 0 ? K <= 4096 : K % 64 == 0 || K <= 1536 || std::min(M, N) <= 128;
}

// Products that k_gemm_nt_direct takes: at most one 32 x 32 tile per CU, at most one round of loads per wave.  Measured
// with a launch behind a launch against the LDS-staged kernels: 197 x 768 x 768 5.1 us for 6.5, 1 x 3072 x 768 4.6 for
// 6.5, 512 x 512 x 512 5.2 for 5.6; but 197 x 3072 x 768 7.8 for 6.8 and 197 x 768 x 3072 (three rounds) 11.5 for 11.1:
// every load instruction touches 32 rows.
inline bool direct_fits(int64_t M, int64_t N, int64_t K) {
    return K >= 16 && K <= 1024 && ((M + 63) / 64) * ((N + 63) / 64) <= 64;
}

// ---- weight gradients of convolutions without stored patches (fxp_conv_wgrad.hip) ----
constexpr int kWgradStep = 128;                       // pixels of a stage
struct WgradCut {
    int bm, tiles_m, tiles_n, slices;
    bool pairs;              // two workgroups per CU
    int64_t per_slice;
    size_t ws_bytes;
};

inline WgradCut plan_conv_wgrad(int64_t M, int64_t Cout, int64_t K) {
    WgradCut p;
    p.bm = Cout <= 64 ? 64 : 128;
    p.tiles_m = static_cast<int>((Cout + p.bm - 1) / p.bm);
    p.tiles_n = static_cast<int>((K + 127) / 128);
    const int64_t tiles = static_cast<int64_t>(p.tiles_m) * p.tiles_n;
    // The number of slices whose rounds take least: eight waves and four stages, one workgroup per CU, 0.75 us a step (0.58 with 64
    // channels), or four waves of 64 x 64 and two stages, two workgroups per CU, 1.25 us a step of both; 4.5 us around the steps; the
    // slices written and read again at 4.5 TB/s, partly under the product that their sum rides with.  More than 64 slices only where
    // they are no more bytes than stored patches would be: few weights, many pixels, and with 64 workgroups at work one tile took
    // longer than patches and their product (steps in us, stored / 64 slices at most / so: 256 x 56 x 56 x 16 -> 96 1x1 273 / 335 / 268,
    // 16 -> 16 151 / 172 / 140, 64 x 56 x 56 x 64 -> 64 1x1 83 / 85 / 76).
    int64_t splits = 1;
    double best = 0.0;
    p.pairs = false;
    for (int pairs = 0; pairs <= (p.bm == 128 ? 1 : 0); ++pairs)
        for (int64_t n = 1; n == 1 || (n <= M / 512 && (n <= 64 || (n <= 512 && 4 * n * Cout <= M))); n += n < 64 ? 1 : 32) {
            if (pairs && tiles * n <= 256) continue;
            const int64_t slots = pairs ? 512 : 256, steps = (M + n * kWgradStep - 1) / (n * kWgradStep);
            const double step_us = pairs ? 1.25 : p.bm == 128 ? 0.75 : 0.58;
            const double us = static_cast<double>((tiles * n + slots - 1) / slots) * (step_us * static_cast<double>(steps) + 4.5) +
                              (n > 1 ? 1.0 + 1.2 * 4.0 * static_cast<double>(n * Cout * K) / 4.5e6 : 0.0);
            if (best == 0.0 || us < best) {
                best = us;
                splits = n;
                p.pairs = pairs != 0;
            }
        }
    if (M > kMaxContraction) splits = std::max<int64_t>(splits, (M + kMaxSlice - 1) / kMaxSlice);
    p.per_slice = ((M + splits - 1) / splits + kWgradStep - 1) / kWgradStep * kWgradStep;
    p.slices = static_cast<int>((M + p.per_slice - 1) / p.per_slice);
    p.ws_bytes = p.slices > 1 ? static_cast<size_t>(p.slices) * ((Cout * K + 3) / 4 * 4) * sizeof(int32_t) : 0;
    return p;
}

// Weight gradients of 1x1 layers that go through stored patches all the same, which are one transposed copy of the image: some 500 to
// 1000 pixels are one slice of five to eight stages, one after the other, but one round of loads of k_gemm_nt_direct (backward
// passes for dW alone, replayed from a graph, stored / from the image in us: 784 pixels 272 -> 400 13.0 / 16.4, 16 -> 32 11.8 / 12.5;
// 960 pixels 512 -> 512 13.2 / 15.7; 576 pixels 128 -> 256 12.3 / 12.6, 256 -> 64 12.1 / 11.5; 512 pixels 128 -> 256 12.5 / 11.9).  Off
// the 16-byte grid that product and the map of dY are slower, and outputs of up to 64 channels stay: whole quads are ahead later the
// more channels there are (700 pixels 16 -> 512 13.2 / 15.3, 128 -> 512 14.7 / 14.5; 900 pixels 128 -> 512 15.3 / 15.5, both gradients
// 512 -> 400 21.9 / 20.6; 980 pixels 512 -> 128 14.3 / 15.5), other counts with the fewest (961 pixels 16 -> 480 15.2 / 16.7, 512 ->
// 256 17.3 / 15.7).
inline bool one_tap_patches(int64_t M, int64_t Cout, int64_t C) {
    if (!direct_fits(Cout, C, M)) return false;
    if (M % 16 == 0) return M > (Cout > 64 ? 512 : 640);
    if (Cout <= 64) return false;
    if (M % 4 == 0) return M > (C <= 32 ? 512 : C <= 256 ? 768 : 960);
    return C == 16 && M > 768;
}

}  // namespace fxp
