// How sums of slices are cut up: host arithmetic only, so that it can be checked without a device.
#pragma once
#include <cstdint>

namespace fxp {

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

}  // namespace fxp
