// Random words of the path tracer: Philox4x32-10 streams, read by word position.  No device
// code of its own, so that it compiles (and is tested) on the host alone.
#pragma once
#include <stdint.h>

#include <type_traits>

namespace ds {

// Counter-based generator of Salmon et al. (SC'11): 10 rounds of two 32x32->64-bit
// multiplications mixing the four counter words, with a Weyl-sequence key schedule.
__host__ __device__ __forceinline__ void philox(uint32_t a, uint32_t b, uint32_t x0, uint32_t x1,
                                                uint32_t x2, uint32_t x3, uint32_t (&out)[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = (uint64_t)0xD2511F53u * x0, m1 = (uint64_t)0xCD9E8D57u * x2;
        const uint32_t y0 = (uint32_t)(m1 >> 32) ^ x1 ^ a, y2 = (uint32_t)(m0 >> 32) ^ x3 ^ b;
        x0 = y0;
        x1 = (uint32_t)m1;
        x2 = y2;
        x3 = (uint32_t)m0;
        a += 0x9E3779B9u;
        b += 0xBB67AE85u;
    }
    out[0] = x0;
    out[1] = x1;
    out[2] = x2;
    out[3] = x3;
}

enum PathKind {
    kRecordPaths,  // L_i (or L_s) of a record: ds_trace_li's estimates
    kPixelPaths,   // path-traced camera samples
    kFirstHits,    // first collision of a camera ray and its direct light
    kRecordDraws,  // record configurations (Sec. 5.1)
};

// A position in a path's stream, in words.  A path takes at most 2^26 tentative collisions of two
// words and as many scatterings of four, far below 2^32.  A record draw retries up to 10^6
// times on one stream, each try a walk of its own, and passes 2^32 words in a nearly empty,
// optically thick grid.
template <int KIND>
using WordPos = typename std::conditional<KIND == kRecordDraws, uint64_t, uint32_t>::type;

// Words 4 block .. 4 block + 3 of stream (id0, id1): counter words 2 and 3 count the blocks.
template <class Pos>
__host__ __device__ __forceinline__ void stream_block(uint64_t seed, uint32_t id0, uint32_t id1, Pos block,
                                                      uint32_t (&out)[4])
{
    philox((uint32_t)seed, (uint32_t)(seed >> 32), id0, id1, (uint32_t)block,
           (uint32_t)((uint64_t)block >> 32), out);
}

}  // namespace ds
