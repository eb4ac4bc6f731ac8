// order.h -- argument block and launcher of the spatial storage order of a
// map (Morton cells, stable radix ranking, brick interleave).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gsr {

// keys per block of a radix pass: 1024 (four rounds of 256 threads), or 4096
// past GSR_RADIX_SMALL keys, where the blocks' counts would outgrow their scan.
// A pass's scatter at 30,011 keys took 15.6 us with 8 blocks of 4096, now 6.6
// with 30 of 1024; at 1M 17.5 and 10.5.
#define GSR_RADIX_SMALL (1 << 20)
static inline int64_t radix_tile(int64_t n) { return n <= GSR_RADIX_SMALL ? 1024 : 4096; }
#define GSR_RADIX_BITS 8     // digit width; four passes cover the 31-bit codes
#define GSR_BOX_BLOCKS 256   // blocks of the box pass, one partial box each

// Workspace: two (code, value) buffers of n entries, the radix counts
// [256][blocks], the digit totals and the partial boxes.
struct OrderArgs {
    int64_t n;
    const float* mean;   // [3][n]
    uint32_t* box;       // [GSR_BOX_BLOCKS][8]: order-preserving images of lo x, y, z, then hi x, y, z
    uint32_t* code[2];   // [n] each: keys, ping-pong between passes
    uint32_t* val[2];    // [n] each: Gaussian indices, ping-pong
    uint32_t* hist;      // [256][blocks]: per-block digit counts, then their offsets within the digit
    uint32_t* tot;       // [256]: keys per digit of the pass
    int32_t blocks;      // radix tiles
    int32_t tile;        // radix_tile(n) keys each
    int32_t brick;
    int64_t full;        // n / brick
    int64_t mult;        // the brick multiplier P
    int32_t* index;      // [n] out
};

hipError_t launch_spatial_order(const OrderArgs& a, hipStream_t s);

}  // namespace gsr
