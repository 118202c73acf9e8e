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

// ---- Fixed-length calls: the kernels with one wave per SIMD (blocks of 256 rows, one per CU) or the 4-wave ones (128
// rows, two per CU).  b = blocks of 256 rows in the launch.  Measured over N = 512 ... 16384 and b = 8 ... 1536, as time of
// the first over time of the second:
//   b <= 128           half the chip idles: forward, d = 128, N = 8192 1.08 ... 1.19 (1.21 ... 1.25 under the mask)
//   128 < b <= 256     one round either way, and a large block beats two small ones: 0.75 ... 0.87 without the mask
//   256 < b <= 384     the last round is at most half full, and small blocks spread over it: d = 128 0.98 ... 1.05, d = 64
//                      1.05 ... 1.30
//   beyond             full rounds: 0.8 ... 0.95 where the key loop outweighs a lone block's prologue
// Under the mask a round's length is that of its unluckiest CU.  A CU's two small blocks are 32 places apart in an XCD's
// list: where 32 is a multiple of a head's tiles (N = 1024, 2048, 4096) those are two tiles of the same length, and the
// CU with the two longest ends last (b = 160, d = 128, forward, N = 2048 ... 8192: 0.94, 1.10 at 3072, 0.89, 0.97, 1.01).
inline bool equal_pairs(int N) { return 32 % (N / 128) == 0; }

inline bool fwd_one_wave(int d_qk, bool causal, int N, long long b)
{
    if (N % 256 != 0 || N < 1024 || b <= 128) return false;
    const bool one_round = b <= 256;
    if (!causal) {          // d = 64: the vector port binds, the gain is smaller (N = 1024 one round 1.01 ... 1.04)
        if (d_qk == 64) return one_round ? N > 1024 : b > 384 && N >= 8192;
        return one_round || N >= 2048;
    }
    if (d_qk == 64)         // (N = 8192, b = 288 ... 384: 0.88, 0.92, 1.03, 0.89; N = 12288 there 1.05 ... 1.10)
        return !one_round && (N >= 16384 || (b <= 384 && N >= 8192 && N < 12288));
    if (one_round) return (equal_pairs(N) && N >= 2048) || (d_qk == 192 && N >= 8192);     // (d = 192, N = 8192: 0.91)
    return N >= (d_qk == 192 ? 6144 : 8192);        // (N = 4096, b = 288 ... 512: 1.02 ... 1.13, at 192 0.98 ... 1.08)
}

// dQ with 64 queries per wave (d_qk = d_v = 128 or 64).
inline bool dq_one_wave(int d_qk, bool causal, int N, long long b)
{
    if (N % 256 != 0 || N < 1024 || b <= 128) return false;
    const bool one_round = b <= 256;
    // (causal, b = 264 ... 512: N = 1024 1.33 ... 0.96, N = 2048 1.24 ... 0.96, N = 1280 and 1536 1.03 ... 0.91)
    if (d_qk == 128) return one_round || !causal || N >= 3072 || !equal_pairs(N);
    if (!causal) return one_round || N >= 2048;
    return one_round ? equal_pairs(N) && N >= 2048 : N >= 8192;            // (N = 1024, b = 264 ... 480: 1.12 ... 1.62)
}

// dK/dV with 64 keys per wave (d = 64); b counts 256-key blocks.
inline bool dkdv64_one_wave(bool causal, int N, long long b)
{
    if (N % 256 != 0 || N < 1024 || b <= 128) return false;
    const bool one_round = b <= 256;
    if (!causal) return one_round || (b > 384 && N >= 2048);               // (N = 8192, b = 288 ... 384: 1.13 ... 1.04, 416: 0.86)
    return one_round ? equal_pairs(N) : N >= 8192;                         // (N = 1024, b = 264 ... 480: 1.06 ... 1.57)
}

// d = 256, the pipelined kernels with one wave per SIMD against the general ones (one block of 128 rows per CU both):
// 0.65 ... 0.97 but for single-tile sequences in more than half a round (N = 128, 128 ... 1024 blocks: dK/dV 1.02 ...
// 1.09, dQ 1.01 ... 1.05 under the mask and 0.87 ... 0.95 without).
inline bool dq256_one_wave(bool causal, int N, long long heads) { return !(causal && N == 128 && heads >= 128); }
inline bool dkdv256_one_wave(int N, long long heads) { return !(N == 128 && heads >= 128); }

}  // namespace attn
