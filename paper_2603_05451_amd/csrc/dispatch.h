// Which block takes which work and which kernel takes which call: arithmetic on sizes alone, without HIP, so that a
// host compiler can build it for a test.
#pragma once
#include <stdint.h>

#if defined(__HIP__)
#define ATTN_ANYWHERE __host__ __device__ __forceinline__
#else
#define ATTN_ANYWHERE inline
#endif

namespace attn {

// Place of a block in the work list (head by head, and within a head table entry by table entry) for kernels whose
// blocks take two 128-row tiles and have nothing to do for every second entry of a sequence.  Blocks are dealt to the
// 8 XCDs round robin; an XCD takes one section of the list, so that tiles of one head share its L2, and in it places
// 0, 2, 4, ... first, then 1, 3, 5, ...: dispatched alternately, the empty blocks would all fall to the same shader
// engines and leave the others twice the work.  The order is one of the section, not of the head: with a head's even
// places before its odd ones, 2 or 4 heads left half of the XCDs with empty blocks alone (d = 64, 16 sequences of
// 4096 tokens, H = 8/2, no mask, dK/dV: 731 us of a 2791 us backward pass).
ATTN_ANYWHERE int section_order(int block, int total)
{
    const bool dealt = (total & 7) == 0;
    const int n = dealt ? total >> 3 : total, p = dealt ? block >> 3 : block, half = (n + 1) >> 1;
    return (dealt ? (block & 7) * n : 0) + (p < half ? 2 * p : 2 * (p - half) + 1);
}

}  // namespace attn
