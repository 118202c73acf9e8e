// Plan tables of the variable-length entry points (paper Sec. 3.3: variable sequence lengths are
// served longest first, after a preprocessing kernel that sorts the batch).
//
// Input: cu_q[0..B] and cu_k[0..B] (device), the running token counts of the packed query-side
// and key-side tensors: sequence b owns query rows cu_q[b] .. cu_q[b+1]-1 and key rows
// cu_k[b] .. cu_k[b+1]-1 (cu_k may be the same array: self-attention).
// Output: two tables, one entry per 128-row QUERY tile and one per 128-row KEY tile.  An entry is
// two int4: {first query row, query length, first key row, key length} of the sequence and
// {tile index inside the sequence, kPlanUsed, sequence index, 0}.  Sequences are ordered by the length of the loop one
// of their tiles runs -- the key tile count for query tiles, the query tile count for key tiles --
// longest first (a counting sort over tile counts; ties keep no particular order, which does not
// matter because no result depends on which block computes which tile), and inside a sequence
// from the last tile to the first (under a causal mask the last query tile has the longest key
// loop; the dK/dV kernels read the index backwards for the same reason).  Unused entries up to
// the table size are zero, except in a table of query tiles with no more queries than sequences: there
// every query of a tile but its first has an entry {the tile's entry, query within the tile, 0, 0}, {0, kPlanHelp,
// 0, 0} behind the used ones, for the decode and merge kernels, and the tile's own entry ends with 1.  The kernels size their grids by the table sizes, host-side upper
// bounds, because the host never reads the lengths; for the same reason the boundaries are checked
// here, on the device, against the row counts the caller stated: a sequence that does not lie
// inside the tensors is left out of both tables.
#include "common.h"
#include "launch.h"

namespace attn {

constexpr int PLAN_NT = 1024;
constexpr int PLAN_BUCKETS = 4096;      // loop lengths 0 .. 4095 tiles; longer ones share the top bucket

// What the kernel costs is its chain of dependent steps -- every packed call waits for it, and a small one takes
// 15-20 us in all.  So: a block per table, boundaries read once into registers (sequences beyond one per thread
// are read again), a scan by wave shuffles with two barriers, and zeros only behind the last entry.
// own/other: the side whose tiles are listed and the side they loop over.
__device__ void plan_build(const int* __restrict__ cu_q, const int* __restrict__ cu_k, int B, int Tq, int Tk, bool own_is_q,
                           int4* __restrict__ plan, int max_tiles)
{
    __shared__ int hist[PLAN_BUCKETS];       // tiles per bucket, then next free entry per bucket
    __shared__ int wave_sum[PLAN_NT / 64];
    __shared__ int next_free;                // first entry that no tile and no helper has taken
    const bool spread = own_is_q && Tq <= B;
    static_assert(PLAN_BUCKETS == 4 * PLAN_NT, "four buckets per thread in the scan below");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto tiles = [](int len) { return (len + 127) / 128; };
    struct Sequence { int qs, ql, ks, kl, nt, key; };
    auto load = [&](int b) {
        Sequence s;
        s.qs = cu_q[b]; s.ql = cu_q[b + 1] - s.qs;
        s.ks = cu_k[b]; s.kl = cu_k[b + 1] - s.ks;
        // A sequence whose rows do not lie inside the tensors (boundaries that decrease, or that run past
        // the totals the caller stated) gets no tiles at all: nothing of it is read or written.  Query tiles
        // of a sequence without keys are not listed.
        const bool inside = s.qs >= 0 && s.ql >= 0 && s.qs <= Tq - s.ql && s.ks >= 0 && s.kl >= 0 && s.ks <= Tk - s.kl;
        s.nt = !inside ? 0 : own_is_q ? (s.kl > 0 ? tiles(s.ql) : 0) : tiles(s.kl);
        const int loop = tiles(own_is_q ? s.kl : s.ql);
        s.key = loop < PLAN_BUCKETS ? loop : PLAN_BUCKETS - 1;
        return s;
    };
    Sequence own = {};
    if (tid < B) own = load(tid);
#pragma unroll
    for (int e = 0; e < 4; ++e) hist[4 * tid + e] = 0;
    __syncthreads();
    if (own.nt > 0) atomicAdd(&hist[own.key], own.nt);
    for (int b = tid + PLAN_NT; b < B; b += PLAN_NT) {
        const Sequence s = load(b);
        if (s.nt > 0) atomicAdd(&hist[s.key], s.nt);
    }
    __syncthreads();
    // Exclusive prefix sum of the tile counts over the buckets from the longest loop down.
    // Position p = 0 .. PLAN_BUCKETS-1 stands for bucket PLAN_BUCKETS-1-p; every thread owns four
    // consecutive positions.
    int w[4], local = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) { w[e] = hist[PLAN_BUCKETS - 1 - (4 * tid + e)]; local += w[e]; }
    int scan = local;                        // inclusive, within the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int below = __shfl_up(scan, off);
        if (lane >= off) scan += below;
    }
    if (lane == 63) wave_sum[wave] = scan;
    __syncthreads();
    int run = scan - local, total = 0;
#pragma unroll
    for (int v = 0; v < PLAN_NT / 64; ++v) {
        const int sum = wave_sum[v];
        if (v < wave) run += sum;
        total += sum;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        hist[PLAN_BUCKETS - 1 - (4 * tid + e)] = run;
        run += w[e];
    }
    // (boundaries that overlap can list more tiles than the table holds, or than an int counts)
    total = min(max(total, 0), max_tiles);
    if (tid == 0) next_free = total;
    if (spread)                              // before the helpers' entries
        for (int i = 2 * total + tid; i < 2 * max_tiles; i += PLAN_NT) plan[i] = make_int4(0, 0, 0, 0);
    __syncthreads();
    // the entries: a sequence's own lane writes them one by one, or the wave 64 at a time, then one sequence after the
    // other.  The lanes take sequences of up to `few` tiles, at least as many as there are longer ones then (both tables, us,
    // all by lanes, all longer than two tiles by the wave, this: 40 x 257 tokens 7.3, 9.4, 3.2; 1500 x 300 20, 32, 8.9;
    // 16 of 64 ... 8192 15, 5.0, 4.4; 3 x 30 000 37, 4.2, 4.3).
    auto entry = [&](int at, int4 rows, int4 tile) {
        if (at < 0 || at >= max_tiles) return;
        plan[2 * at] = rows;
        plan[2 * at + 1] = tile;
    };
    auto put = [&](const Sequence& s, int b) {
        int first = 0, few = 2, helper = 0, helped = 0;
        if (s.nt > 0) first = atomicAdd(&hist[s.key], s.nt);
        if (spread && s.nt > 0 && s.ql > s.nt) {
            helper = atomicAdd(&next_free, s.ql - s.nt);
            helped = helper >= total && helper <= max_tiles - (s.ql - s.nt);
        }
        while (few < 64 && __popcll(__ballot(s.nt > few)) > few) few *= 2;
        if (s.nt > 0 && s.nt <= few)
            for (int t = 0; t < s.nt; ++t)
                entry(first + t, make_int4(s.qs, s.ql, s.ks, s.kl), make_int4(s.nt - 1 - t, kPlanUsed, b, helped));
        auto each = [&](bool mine, auto f) {     // f(l) by the whole wave, for every lane l with `mine`
            for (uint64_t left = __ballot(mine); left; left &= left - 1) f(__builtin_ctzll(left));
        };
        auto of = [&](int x, int l) { return __builtin_amdgcn_readlane(x, l); };
        each(s.nt > few, [&](int l) {
            const int nt = of(s.nt, l), at = of(first, l), sb = of(b, l), h = of(helped, l);
            const int4 rows = make_int4(of(s.qs, l), of(s.ql, l), of(s.ks, l), of(s.kl, l));
            for (int t = lane; t < nt; t += 64) entry(at + t, rows, make_int4(nt - 1 - t, kPlanUsed, sb, h));
        });
        if (spread)
            each(helped != 0, [&](int l) {
                const int ql = of(s.ql, l), last = of(first, l) + of(s.nt, l) - 1, at = of(helper, l) - 1;
                for (int i = lane; i < ql; i += 64)
                    if (i % 128) entry(at + i - i / 128, make_int4(last - i / 128, i % 128, 0, 0), make_int4(0, kPlanHelp, 0, 0));
            });
    };
    put(own, tid);
    for (int b0 = PLAN_NT; b0 < B; b0 += PLAN_NT) put(b0 + tid < B ? load(b0 + tid) : Sequence{}, b0 + tid);
    if (!spread)
        for (int i = 2 * total + tid; i < 2 * max_tiles; i += PLAN_NT) plan[i] = make_int4(0, 0, 0, 0);
}

// Block 0: the table of query tiles; block 1 (backward only): the table of key tiles.
__global__ void __launch_bounds__(PLAN_NT)
varlen_plan_kernel(const int* __restrict__ cu_q, const int* __restrict__ cu_k, int B, int Tq, int Tk,
                   int4* __restrict__ plan_q, int max_tiles_q, int4* __restrict__ plan_k, int max_tiles_k)
{
    const bool queries = blockIdx.x == 0;
    plan_build(cu_q, cu_k, B, Tq, Tk, queries, queries ? plan_q : plan_k, queries ? max_tiles_q : max_tiles_k);
}

int launch_varlen_plan(const int* cu_q, const int* cu_k, int B, int Tq, int Tk, void* plan_q, int max_tiles_q,
                       void* plan_k, int max_tiles_k, void* stream)
{
    return launch_kernel(varlen_plan_kernel, dim3(plan_k ? 2 : 1), dim3(PLAN_NT), 0, stream, cu_q, cu_k, B, Tq, Tk,
                         (int4*)plan_q, max_tiles_q, (int4*)plan_k, max_tiles_k) == hipSuccess ? 0 : -3;
}

}  // namespace attn
