// seed_lanes.h -- how many lanes triangulate a pixel.
#pragma once
#include <stdint.h>

namespace gsr {

// One lane per neighbour up to four (1000 pixels, four neighbours: 69 us with
// one lane, 24 with four; 500k: the same), and never more than a launch holds:
// a grid's threads are counted in 32 bits, whole blocks of 256, so the four
// lanes halve past 2^30 - 64 pixels and the two past 2^31 - 128.
static inline int seed_lanes(int64_t n, int32_t neighbours)
{
    int lanes = neighbours >= 3 ? 4 : (neighbours == 2 ? 2 : 1);
    while (n * lanes > (1ll << 32) - 256) lanes /= 2;
    return lanes;
}

}  // namespace gsr
