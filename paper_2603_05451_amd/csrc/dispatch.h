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

// Place of a block in the work list of a launch over tables whose blocks take two 128-row tiles and have nothing to do for every
// second entry of a sequence.  An XCD takes one section of the list, and in it places 0, 2, 4, ... first, then 1, 3, 5, ...:
// dispatched alternately, the empty blocks would all fall to the same shader engines and leave the others twice the work.
// The order is one of the section, not of the head: with a head's even places before its odd ones, 2 or 4 heads left half of
// the XCDs with empty blocks alone (d = 64, 16 sequences of 4096 tokens, H = 8/2, no mask, dK/dV: 731 us of a 2791 us backward
// pass).
ATTN_ANYWHERE int even_before_odd(int p, int n)
{
    const int half = (n + 1) >> 1;
    return p < half ? 2 * p : 2 * (p - half) + 1;
}
ATTN_ANYWHERE int section_order(int block, int total)
{
    const bool dealt = (total & 7) == 0;
    const int n = dealt ? total >> 3 : total;
    return (dealt ? (block & 7) * n : 0) + even_before_odd(dealt ? block >> 3 : block, n);
}

// ---- Order of the blocks of a launch over heads x tiles (a head's tiles listed longest first, or as a table lists them).
// Blocks are dealt to the 8 XCDs round robin.  An XCD works on heads of its own, one after the other, so that the tiles of a
// head share its L2.  Where the heads do not divide and the tiles are not alike, 2, 4 or 8 XCDs work on a unit of heads together
// and take its places in turn: in contiguous shares (the longer tiles of a head here, the shorter there) the first XCD ends last
// (packed batch of 16 sequences of 64 ... 8192 tokens under the mask, H = 16/4, d = 128, four KV heads on eight XCDs: backward
// pass 2237 us, 1917 in turn).  Every second turn is taken in reverse: the first XCD does not get the longer tile each time, nor one
// of them all places of the parity that is empty in kernels which take two entries per block.
// Under the causal mask the tiles of a group of heads are taken together, longest first: one head's tiles after
// the other's end with the longest tiles of the last head beside idle CUs, and pair long with short ones on a
// CU at random.  (Forward / dQ / dK/dV, us, head by head -> groups of 8: B = 16, H = 16, N = 1024, d = 128: 106 -> 92, 170 -> 158,
// 211 -> 188; B = 4, H = 8, N = 2048, d = 256, a unit of 4 heads: 132 -> 97, 133 -> 110, 233 -> 183; N = 8192, d = 128, H = 16,
// B = 2: 476 -> 457, 650 -> 632, 943 -> 927.)
// Where nothing is to be balanced -- equal tiles without the mask, or a launch of at most one block per CU, which ends with its
// longest tile in any order -- an XCD takes a contiguous share of the places, head by head: in a unit of many heads it reads the
// rows of all of them (us, units -> shares as before: no mask, 31 heads of N = 1024 forward d = 96 21.5 -> 17.8, d = 128 24.5 ->
// 21.3, d = 256 45 -> 40, its backward pass 150 -> 131; 15 of 4096, d = 64 87.8 -> 80.0; mask, 13 of 2048, (192, 128) 51.0 -> 48.3,
// d = 96 backward pass 86.4 -> 80.9; beyond 256 blocks the mask needs the units: 12 of 4096, d = 64 48 against 68).
struct TileOrder {
    int dealt;          // whether every XCD gets an eighth of the places; otherwise they go by the block's number
    int unit, log_m;    // `unit` heads are worked on by 2^log_m XCDs
    int group;          // heads whose tiles are taken together
    int share;          // places of an XCD in a row, before those of the next; 0: by units
    // `own` heads of an XCD's own behind its `first` places of the units, taken together in groups of `own_group`
    int own, first, own_group;
};
struct Place {
    int xcd, at;        // at: in the XCD's list
};
struct HeadTile {
    int head, tile;
};

inline TileOrder tile_order(int heads, int tiles)
{
    const int64_t total = (int64_t)heads * tiles;
    const bool dealt = (total & 7) == 0;
    int log_m = 0;
    if (dealt) while (((int64_t)heads << log_m & 7) != 0) ++log_m;
    return {dealt, dealt ? (int)(((int64_t)heads << log_m) >> 3) : heads, log_m, 1, 0, 0, 0, 0};
}
// The same in contiguous shares.
inline TileOrder share_order(int heads, int tiles)
{
    const TileOrder o = tile_order(heads, tiles);
    return o.log_m == 0 ? o : TileOrder{1, 0, 0, 1, (int)((int64_t)heads * tiles >> 3), 0, 0, 0};
}

// The same under the causal mask.  `share` heads read the same rows, `bytes` of them.  Groups of about 8 heads (4 ... 16 are
// within 3 % of each other) whose rows are no more than 16 MB: all the blocks of a group walk along them at once, and where
// they drift apart the L2 no longer holds what they share (N = 16384, d = 128, 8 MB per head, B = 4, H = 16: dK/dV 7586, 7508,
// 7632, 7958 us in groups of 1, 2, 4, 8).  Equal groups: a small last one ends like a single head (12 heads, N = 1024,
// d = 256, forward: 102 us one by one, 88 as 8 + 4, 80 as 12).
// From 32 heads on, and from 17 where the unit would be all of them, an XCD has heads enough of its own: only those left over
// are shared in units, before its own, and it does not read the rows of every head of a large unit (us, units -> this, in brackets
// contiguous shares: forward, 63 heads of N = 1024, d = 96 31.2 -> 23.5 (26.8), d = 128 37.2 -> 28.2 (32.3); 47 of 2048, d = 128 83 ->
// 61 (79); 100 of 512, d = 96 18.2 -> 13.9 (16.7); 25 of 2048, d = 192 68 -> 53, its backward pass 172 -> 133; 17 of 4096, d = 128
// 102 -> 84.  Fewer: 15 of 4096, forward, d = 96 66 -> 79, d = 256 209 -> 155; 20 of 4096, d = 64 61 -> 66, d = 128 93 -> 97; 28 of 2048
// 0.99 ... 1.03).
inline TileOrder causal_order(int heads, int tiles, int share, int64_t bytes)
{
    TileOrder o = tile_order(heads, tiles);
    if (o.log_m > 0 && (int64_t)heads * tiles <= 256) return share_order(heads, tiles);
    const int64_t fit = (16 << 20) / (bytes < 1 ? 1 : bytes), most = (fit < 1 ? 1 : fit) * share;
    const int want = (int)(most < 8 ? most : 8);
    auto groups = [&](int unit) { const int n = unit / want < 1 ? 1 : unit / want; return (unit + n - 1) / n; };
    if (o.log_m > 0 && heads >= (o.log_m == 3 ? 17 : 32)) {
        const int own = heads / 8;
        o = tile_order(heads - 8 * own, tiles);
        o.own = own;
        o.first = o.unit * tiles >> o.log_m;
        o.own_group = groups(own);
        o.group = o.unit;
        return o;
    }
    o.group = groups(o.unit);
    return o;
}

// Order and blocks of a launch over query tiles (forward, dQ) or key tiles (dK/dV) of `rows` rows (FwdArgs, BwdArgs).
// Equal-length batches count every (sequence, head) as a head; the tables of packed ones are sorted already, for every head
// alike, and list 128-row tiles whatever `rows`.  In a launch of 256-row blocks over equal lengths every block has work: were
// 128-row tiles its places, an XCD's list would have to keep the empty ones from alternating with the live ones, which
// under the mask, where places go from head to head of a group, no order of places does (dQ, d = 128, B H = 32 heads in groups of
// 4, N = 4096: two empty places, two live ones, and so on).
template <typename Args>
inline int tiles_of_query_launch(const Args& a, int rows)
{
    return a.max_tiles == 0 ? a.N / rows : a.st.nq > 0 ? (a.st.nq + rows - 1) / rows : a.max_tiles;
}
template <typename Args>
inline int tiles_of_key_launch(const Args& a, int rows)
{
    return a.max_tiles == 0 ? a.N / rows : a.st.nq > 0 ? (a.st.nk + rows - 1) / rows : a.max_tiles_k;
}
template <typename Args>
inline int query_blocks(const Args& a, int rows) { return tiles_of_query_launch(a, rows) * (a.max_tiles > 0 && a.st.nq == 0 ? 1 : a.B) * a.H; }
template <typename Args>
inline int key_blocks(const Args& a, int rows) { return tiles_of_key_launch(a, rows) * (a.max_tiles > 0 && a.st.nq == 0 ? 1 : a.B) * a.Hkv; }

template <typename Args>
inline TileOrder query_order(const Args& a, int rows)
{
    const int tiles = tiles_of_query_launch(a, rows);
    if (a.max_tiles > 0 && a.st.nq == 0) return tile_order(a.H, tiles);
    if (!a.causal) return share_order(a.B * a.H, tiles);
    return causal_order(a.B * a.H, tiles, a.H / a.Hkv, (int64_t)(a.max_tiles > 0 ? a.st.nk : a.N) * (a.d_qk + a.d_v) * 2);
}
template <typename Args>
inline TileOrder key_order(const Args& a, int rows)
{
    const int tiles = tiles_of_key_launch(a, rows);
    if (a.max_tiles > 0 && a.st.nq == 0) return tile_order(a.Hkv, tiles);
    if (!a.causal) return share_order(a.B * a.Hkv, tiles);
    // the query heads of a KV head pass one after the other: two of them are in flight where blocks drift apart
    const int in_flight = a.H > a.Hkv ? 2 : 1;
    return causal_order(a.B * a.Hkv, tiles, 1, (int64_t)(a.max_tiles > 0 ? a.st.nq : a.N) * (a.d_qk + a.d_v) * 2 * in_flight);
}

// Whether the dK/dV kernel of one block per CU gets 256 blocks that take an XCD's places in turns (32 apart, every second
// turn in reverse) instead of one block per place.  A block then brings in its next tile under the end of the one before
// (N = 128 ... 1024, 65 536 x 16 rows, d = 128, no mask: 4 ... 10 % of the backward pass, N = 8192 0.5 %; d = 64: dkdv64_one_wave),
// but nobody evens out what the turns leave uneven: under the mask only where they are whole pairs of rounds of short
// sequences (N = 512 -8 %, 1024 and 2048 -2 %, 4096 -1, 8192 0; 12 heads of N = 2176 +16 %, 7 x 12 of 1152 +2).
inline bool takes_turns(const TileOrder& o, int tiles, int64_t items, bool causal)
{
    if (items <= 256) return false;
    return !causal || (o.dealt && o.log_m == 0 && items % 512 == 0 && tiles <= 16);
}

// Place of a block; for launches over tables with nothing to do at every second entry, in the order of section_order.
ATTN_ANYWHERE Place block_place(const TileOrder& o, int block)
{
    return o.dealt ? Place{block & 7, block >> 3} : Place{0, block};
}
ATTN_ANYWHERE Place block_place_alternate(const TileOrder& o, int block, int total)
{
    return o.dealt ? Place{block & 7, section_order(block, total) - (block & 7) * (total >> 3)} : Place{0, section_order(block, total)};
}

// The place of a block of `rows` rows in a launch over equal lengths or over tables of 128-row tiles.
ATTN_ANYWHERE Place entry_place(const TileOrder& o, int rows, bool equal, int block, int total)
{
    return rows == 256 && !equal ? block_place_alternate(o, block, total) : block_place(o, block);
}

// (head, tile) of a place: in the order of share_order; of tile_order; in any.  Three functions, and in the last branches instead
// of divisions by 1: what a block does before its first load it waits for, and an integer division is 0.1 us (two heads of
// N = 128, d = 64, without the mask: dQ and dK/dV kernels 6.0 and 6.7 us with the last function, 5.8 and 6.3 with the first).
ATTN_ANYWHERE HeadTile head_tile_in_shares(const TileOrder& o, Place place, int tiles)
{
    const int p = place.xcd * o.share + place.at, head = p / tiles;
    return {place.xcd * o.unit + head, p - head * tiles};
}
ATTN_ANYWHERE HeadTile head_tile_in_units(const TileOrder& o, Place place, int tiles)
{
    const int m = 1 << o.log_m, turn = place.xcd & (m - 1), p = place.at * m + ((place.at & 1) ? m - 1 - turn : turn), head = p / tiles;
    return {(place.xcd >> o.log_m) * o.unit + head, p - head * tiles};
}
ATTN_ANYWHERE HeadTile head_tile(const TileOrder& o, Place place, int tiles)
{
    const int m = 1 << o.log_m, turn = place.xcd & (m - 1);
    int p = place.xcd * o.share + place.at * m + ((place.at & 1) ? m - 1 - turn : turn);
    int base = (place.xcd >> o.log_m) * o.unit, unit = o.unit, group = o.group;
    if (o.own > 0 && place.at >= o.first) {
        p = place.at - o.first;
        base = (8 >> o.log_m) * o.unit + place.xcd * o.own;
        unit = o.own;
        group = o.own_group;
    }
    if (group == 1) {
        const int head = p / tiles;
        return {base + head, p - head * tiles};
    }
    int first = 0, r = p;
    if (group < unit) {
        const int whole = group * tiles, g = p / whole;
        first = g * group;
        r = p - g * whole;
    }
    const int width = unit - first < group ? unit - first : group, tile = r / width;
    return {base + first + (r - tile * width), tile};
}

// ---- Fixed-length calls: the kernels with one wave per SIMD (blocks of 256 rows, one per CU) or the 4-wave ones (128
// rows, two per CU).  b = blocks of 256 rows in the launch.  Measured over N = 512 ... 16384 and b = 8 ... 1536, as time of
// the first over time of the second:
//   b <= 128           half the chip idles: forward, d = 128, N = 8192 1.08 ... 1.19 (1.21 ... 1.25 under the mask)
//   128 < b <= 256     one round either way, and without the mask a large block beats two small ones: 0.75 ... 0.87
//   256 < b <= 384     the last round is at most half full, and small blocks spread over it: d = 128 0.98 ... 1.05, d = 64
//                      1.05 ... 1.30
//   beyond             full rounds: 0.8 ... 0.95 where the key loop outweighs a lone block's prologue
// Under the mask a round's length is that of its unluckiest CU, and with the tiles of a group of heads taken together (causal_order)
// the small blocks of a CU are a long and a short one: in one round the large blocks, each alone on its CU, end with the longest.
inline bool fwd_one_wave(int d_qk, bool causal, int N, long long b)
{
    if (N % 256 != 0 || N < 1024 || b <= 128) return false;
    const bool one_round = b <= 256;
    if (!causal) {          // d = 64: the vector port binds, the gain is smaller (N = 1024 one round 1.01 ... 1.04)
        // (N = 4096 ... 6144, rounds 15/16 full: b = 480 and 512 0.92 ... 0.95, 960 and 1024 0.92 ... 0.96, 2048 0.95 and 0.96, 4096
        // 1.00; 7/8 full: 448 0.92, 896 1.03; N = 3072 0.98 ... 1.03, 2048 1.01 ... 1.06, 1024 1.03 ... 1.13)
        if (d_qk == 64) return one_round ? N > 1024 : b > 384 && (N >= 8192 || (N >= 4096 && b >= (b + 255) / 256 * 240));
        return one_round || N >= 2048;
    }
    // d = 64: one round 1.30 ... 1.42; N = 4096 ... 8192, b = 288 ... 384 1.04 ... 1.16, two full rounds (432 ... 528) 0.92 ... 0.97 from
    // N = 8192 (1.00 at 4096), 576 ... 768 1.02 ... 1.16; N = 16384 from b = 1024 0.98 ... 0.99
    if (d_qk == 64) return N >= 8192 && ((b > 416 && b <= 512) || (N >= 16384 && b >= 1024));
    // d = 128: one round 1.05 ... 1.33.  d = 192, one round: N = 2048 1.08 ... 1.14, N = 3072 1.03 ... 1.10, N = 4096 b <= 192 1.03 ... 1.08,
    // from b = 208 1.02 and 1.01 with even numbers of heads, 0.89 and 0.82 with odd ones, N = 5120 ... 7168 from 200 0.85 ... 1.03, below
    // 1.03 ... 1.05, N = 8192 and more 0.75 ... 1.03
    if (one_round) return d_qk == 192 && N >= (b > 192 ? 4096 : 8192);
    // d = 128: N = 4096, b = 272 ... 352 1.03 ... 1.08, from 384 0.89 ... 1.05 (0.96 on average), N = 5120 from 400 0.88 ... 0.99 (1.13 where
    // the blocks are no multiple of 8), N = 6144 0.87 ... 1.05, N = 3072 0.95 ... 1.13.  d = 192: N = 4096 0.86 ... 1.03, N = 5120 ... 6144
    // 0.82 ... 1.09, N = 3072 0.85 ... 1.02
    return N >= 6144 || (N >= 4096 && (d_qk == 192 || b >= 384));
}

// dQ with 64 queries per wave (d_qk = d_v = 128 or 64).
inline bool dq_one_wave(int d_qk, bool causal, int N, long long b)
{
    if (N % 256 != 0 || N < 1024 || b <= 128) return false;
    const bool one_round = b <= 256;
    if (!causal) return one_round || N >= 2048 || d_qk == 128;
    // (mask, share of the whole backward pass: one round d = 128 0.99 ... 1.05, d = 64 1.04 ... 1.11; beyond, d = 128: N = 1024 ... 1792 b = 288 ...
    // 320 0.99 ... 1.17, from 384 0.96 ... 1.01, N = 2560 and more 0.92 ... 1.00; d = 64: N = 4096 and more b = 288 ... 352 1.00 ... 1.04, from 384
    // 0.94 ... 0.99, N = 1024 ... 3072 0.97 ... 1.14)
    if (one_round) return false;
    return d_qk == 128 ? N >= 2560 || b > 320 : N >= 4096 && b >= 384;
}

// dK/dV with 64 keys per wave (d = 64); b counts 256-key blocks.
inline bool dkdv64_one_wave(bool causal, int N, long long b)
{
    if (N % 256 != 0 || b <= 128) return false;
    // In turns the next tile's first rows come under the end of the one before: no mask, turns at least 7/8 full (share of the
    // whole backward pass: N = 256 ... 1024, b = 448 0.88 ... 0.95, 480 0.94 ... 0.96, 896 ... 960 0.94 ... 0.97, 1024 0.94 ... 0.96,
    // 1856 0.99, 4096 0.94 ... 0.96; b = 264 and 272 1.08 and 1.06, 540 1.04, 576 1.02; N = 2048 and more 0.98 ... 1.00)
    if (!causal && b > 256 && b >= (b + 255) / 256 * 224) return true;
    if (N < 1024) return false;
    const bool one_round = b <= 256;
    if (!causal) return one_round || (b > 384 && N >= 2048);               // (N = 8192, b = 288 ... 384: 1.13 ... 1.04, 416: 0.86)
    return N >= 4096 && b > 384;        // (mask: one round 1.08 ... 1.17, b = 288 ... 384 0.98 ... 1.07, beyond 0.94 ... 1.02, N = 3072 and less 0.98 ... 1.19)
}

// The general kernels at d = 64, three blocks of 4 waves per CU and not two, where there are more blocks than two per CU hold; loop = mean
// number of rows that a block walks.  (Share of the whole backward pass.  Variable length, no mask 0.90 ... 1.00, mask 0.86 ... 1.00; fixed length
// 0.96 ... 1.00 and 0.95 ... 1.00.  Up to 512 blocks 1.00 ... 1.045, and under the mask 528 ... 640 blocks 0.96 ... 1.06: a block alone or beside
// one other misses what the wider kernel reads ahead.  Dk and dV of 700 keys: 60 queries 1.05 (mask 0.97), 100 ... 128 1.01 and 1.02, 130 0.94.)
// Variable length, equal lengths, no mask, just past three blocks per CU, short loops: 300 rows 792 blocks 1.03, 600 rows 776 ... 1000 1.00 ... 1.02, 1040
// 0.96; 640 rows 0.97 ... 1.00, 2000 1.00; under the mask 300 ... 2000 rows 0.89 ... 0.97; fixed length 0.97 ... 0.99.
inline bool lean_blocks(int d_qk, bool causal, long long blocks, long long loop, bool strided = false)
{
    if (strided && !causal && loop <= 600 && blocks > 768 && blocks <= 1024) return false;
    return d_qk == 64 && loop > 128 && blocks > (causal ? 640 : 512);
}
// Tiles of 128 rows in a packed batch, of which the host knows the totals: half a tile per sequence is past its end.  (The tables have room for
// T / 128 + B.  Blocks of 64 ... 300 rows x 64 sequences x 4 heads: 436 by this, 432 there, room for 564, on which three blocks per CU
// took 1.04; 129 ... 1000 x 64 x 2 512, 520, 576, 1.06; 140 ... 500 x 20 x 8 456, 464, 536, 1.06; 200 ... 400 x 24 x 8 536, 520, 632, 0.97.)
inline long long likely_tiles(bool equal, int max_tiles, int T, int B) { return equal ? max_tiles : (long long)T / 128 + B / 2; }
// dQ: not for a single query tile per sequence (no mask / mask, dK and dV on the wide kernel: 60 queries against 700 keys 1.00 / 1.02, 2000 keys
// 1.06 / 1.05; 128 against 700 1.01 / 1.01, 2000 1.05 / 1.04; 129 against 700 0.95 / 0.90, 300 against 2000 0.93 / 0.89).
inline bool lean_dq_blocks(int d_qk, bool causal, long long blocks, long long queries, long long keys, bool strided)
{
    return queries > 128 && lean_blocks(d_qk, causal, blocks, keys, strided);
}

// d = 256, the pipelined kernels with one wave per SIMD against the general ones (one block of 128 rows per CU both):
// 0.65 ... 0.97 but for single-tile sequences in more than half a round (N = 128, 128 ... 1024 blocks: dK/dV 1.02 ...
// 1.09, dQ 1.01 ... 1.05 under the mask and 0.87 ... 0.95 without).
inline bool dq256_one_wave(bool causal, int N, long long heads) { return !(causal && N == 128 && heads >= 128); }
inline bool dkdv256_one_wave(int N, long long heads) { return !(N == 128 && heads >= 128); }

// ---- Equal lengths, few keys: dQ, dK and dV in one kernel (attn_bwd_short_kernel.inc), a block per (sequence, KV head) that holds all its
// keys, of four waves and two per CU up to 128 keys (d = 64: 256), of eight and one per CU beyond.  Share of the two kernels' time:
//   few steps of 32 queries: one launch for two, in every number of blocks: 1 ... 3 steps 0.62 ... 0.88; 4 0.70 ... 0.97 (d = 64, more than
//            256 keys 1.02); 5 0.74 ... 0.82 at d = 96 and 128 with 8 waves (0.80 and 0.88 with 4), 1.03 at d = 64, 6 0.87 ... 1.18
//   more:    a block walks alone along queries that the two kernels spread over many, so it takes blocks enough to fill the chip:
//            d = 64, up to 128 keys, 4 ... 16 steps  128 blocks 0.95 ... 1.29, 224 0.96 ... 1.03, 256 0.82 ... 0.99, 512 0.63 ... 0.66
//            d = 64, 160 keys  160 blocks 0.76 ... 1.04, 224 0.73 ... 0.83; 200 keys  224 0.85 ... 1.01, 256 0.86 ... 0.95; 256 keys  256 0.91 ... 1.08,
//            320 0.78 ... 0.82, 512 0.61 ... 0.79
//            d = 64, up to 512 keys, rounds of 256: ragged 192 blocks 0.81 ... 0.94, 256 0.75 ... 0.90, 320 1.14 ... 1.17, 512 and 1024 0.85 ... 0.92
//            d = 96  up to 128 keys 128 blocks 1.02 ... 1.15, 160 0.89 ... 1.00, 224 0.81 ... 0.90; up to 256 128 0.84 ... 1.15, 160 0.49 ... 0.86, 512 0.59 ... 0.68
//            d = 128 up to 128 keys 160 blocks 0.94 ... 1.28, 192 0.80 ... 1.19, 224 0.70 ... 1.09, 256 0.68 ... 1.06, 512 0.45 ... 0.59; up to 256 128 0.74 ... 1.11, 160 0.45 ... 0.89, 256 0.42 ... 0.76,
//            512 0.53 ... 0.85
//            77 keys against 1000 queries  64 blocks 1.5 ... 1.9, 256 0.85 (d = 64) and 0.90 (128), 1024 0.61 and 0.52: waves without keys
//   just past a round (512 blocks of four waves, 256 of eight), long walks (steps of 32 ... 128): the last blocks run alone
//            d = 64, up to 128 keys 520 and 544 blocks 1.04 ... 1.08 (query heads of a group under the mask 0.99 ... 1.01), 576 0.94 ... 1.06; 160 keys 520
//            0.89 ... 1.00; 192 ... 256 keys 520 1.02 ... 1.14, 544 0.98 ... 1.13, 576 0.94 ... 1.08, 608 0.86 ... 0.99; 1032 0.66 ... 0.81; 256 keys, 16 steps 520
//            1.02 ... 1.05, 544 0.98 ... 1.04; 192 keys also 256 ...
//            288 0.97 ... 1.08, up to 128 keys against 4096 queries 264 1.10, 320 0.97
//            d = 96  up to 128 keys 0.71 ... 0.91; 192 and 256 keys 264 0.96 ... 1.14, 296 0.99 ... 1.10, 320 0.94 ... 1.08, 352 0.84 ... 1.02, 520 0.83 ... 0.93
//            d = 128 up to 128 keys 0.69 ... 0.90; 256 keys, or more than four times as many queries as keys 264 1.00 ... 1.16, 296 1.00 ... 1.12, 320
//            0.94 ... 1.06, 352 0.87 ... 1.03, 520 0.85 ... 0.98; else 264 0.78 ... 0.98
//            d = 64, 300 keys, four rounds and more 776 blocks 1.07 ... 1.11 (2048 queries 0.89), 1032 1.00 ... 1.07 (0.78); 450 keys 776 0.98 ... 1.02
inline int short_keys(int d_qk, int d_v) { return d_qk != d_v ? 0 : d_qk == 64 ? 512 : d_qk <= 128 ? 256 : 0; }
inline bool short_last_round_alone(int d_qk, int nq, int nk, int64_t blocks, int64_t steps)
{
    auto past = [&](int64_t round, int64_t most) { return blocks > round && blocks <= most; };
    if (steps < 32) return d_qk == 64 && nk > 224 && steps >= 16 && past(512, 544);
    if (d_qk == 64) {
        if (nk <= 128) return past(512, 576) || (steps >= 96 && past(256, 288));
        return nk > 160 && (past(512, 576) || (nk <= 208 && past(255, 288)));
    }
    return nk > 128 && past(256, 320) && (nk > (d_qk == 96 ? 160 : 224) || nq >= 4 * nk);
}
// Whole tiles (equal numbers of queries and keys, a multiple of 128): the line of the fixed-length call, whose kernels are faster than the
// variable-length ones, for both, since contiguous tensors get the same bits from both.  The one kernel takes whole rounds, the two as long as
// they have blocks (share of the fixed-length call's two kernels; G query heads per KV head):
//   d = 64, 128 tokens, rounds of 512  mask   G = 2 ... 4 256 0.96 ... 1.01, 512 0.71 ... 0.75, 544 0.87 ... 1.01; G = 8 and 16 320 0.99 and 1.11, 384 0.92 and 1.02,
//                                             512 0.84, 544 1.12 and 1.23, 704 1.01 and 1.05, 768 0.93 and 0.97, 1056 1.00 and 1.02
//                                      none   G = 2 256 1.04, 288 0.92, 544 1.02; G = 4 288 1.02, 320 0.98, 512 0.82, 544 1.13, 768 1.06, 832 0.97, 1152 1.07, 1280 0.98;
//                                             G = 8 and 16 384 1.01 and 1.14, 480 0.95 and 1.05, 544 1.28 and 1.36, 896 0.98 and 1.03, 960 0.95 and 0.98, 1408 0.96 and 0.99
//           256 tokens                 mask   G = 2 320 0.96, 544 1.10, 640 1.02, 704 0.96; G = 4 ... 16 320 1.10 ... 1.22, 384 0.92 ... 0.98, 544 1.25, 704 0.97 ... 1.02, 1056 1.04
//                                      none   G = 1 320 0.94, 512 0.79, 540 1.04, 600 1.00; G = 2 ... 16 384 1.01 ... 1.28, 480 0.93 ... 1.05, 544 1.16 ... 1.42, 896 1.00 ... 1.08, 960 1.00
//           384 and 512, of 256        mask   240 0.83 ... 1.02, 264 1.37 ... 1.70, 480 0.96 ... 1.03, 768 0.90 ... 1.00; none  240 and 256 G = 1, 2 0.88 ... 1.01, G = 4 1.02 ... 1.07,
//                                             512 1.01 ... 1.11, 768 1.04 ... 1.09
//   d = 96, 128 tokens   G = 2 192 0.90; G = 4 192 0.99 ... 1.03, 208 0.93; G = 8 and 16 208 1.01 ... 1.06, 224 0.97 ... 1.02, 264 0.84 ... 1.03, 528 0.91 ... 0.98
//   d = 128              mask or G = 2, 4 224 0.88 ... 0.98; none, G = 8 and 16 224 ... 256 1.07 ... 1.21, 264 0.96 ... 0.99, G = 16 528 1.14, 576 1.08, 640 0.96
//   256 tokens           d = 96 and 128 G = 2, 4 160 0.80 ... 1.03, G = 8, 16 160 0.92 ... 1.15, 176 0.88 ... 1.03; 264 1.00 ... 1.39, 320 0.98 ... 1.24, 352 mask 0.94 ... 1.08, none d = 96
//                        0.94 ... 1.07, d = 128 1.08 ... 1.20, 400 0.87 ... 1.00; d = 128 none 528 1.05 ... 1.12, 576 1.01 ... 1.08, 640 0.97 ... 1.00, other 528 0.91 ... 1.04
inline bool bwd_short_whole(int d, bool causal, int n, int64_t blocks, int64_t steps)
{
    auto past = [&](int64_t round, int64_t most) { return blocks > round && blocks <= most; };
    if (n > 256) {
        const int64_t rounds = (blocks + 255) / 256;
        return blocks >= rounds * 240 && (causal || (rounds == 1 && steps <= 32));
    }
    if (d == 64) {
        const int64_t rounds = (blocks + 511) / 512;
        int percent;                                           // of full rounds
        if (n == 128) percent = causal ? (steps <= 16 ? 50 : 72) : steps <= 8 ? 52 : steps > 16 ? 90 : rounds == 1 ? 60 : 80;
        else percent = steps <= 8 ? 56 : causal ? (steps <= 16 ? 62 : 70) : 90;
        return 100 * blocks >= percent * 512 * rounds;
    }
    if (n == 128) {
        if (d == 96) return blocks >= (steps > 16 ? 224 : steps > 8 ? 208 : 192);
        return blocks >= (causal || steps < 32 ? 224 : 257) && !(!causal && steps >= 64 && past(512, 592));
    }
    const int64_t alone = causal ? 336 : d == 128 ? 384 : steps >= 64 ? 368 : 336;
    return blocks >= (steps >= 48 ? 176 : 160) && !(steps >= 16 && past(256, alone)) && !(d == 128 && !causal && steps >= 16 && past(512, 592));
}
inline bool bwd_short(int d_qk, int d_v, bool causal, int nq, int nk, int B, int H, int Hkv)
{
    if (nk > short_keys(d_qk, d_v)) return false;
    const int64_t blocks = (int64_t)B * Hkv, steps = (int64_t)(H / Hkv) * ((nq + 31) / 32);
    if (steps <= (nk > 256 ? 3 : d_qk == 64 || nk <= 128 ? 4 : 5)) return true;
    if (nq == nk && nq % 128 == 0) return bwd_short_whole(d_qk, causal, nq, blocks, steps);
    if (nk < 96) return blocks >= 1024;
    if (nk > 256) return blocks >= (blocks + 255) / 256 * (nk <= 384 && steps < 32 && blocks > 768 ? 240 : 192);
    if (short_last_round_alone(d_qk, nq, nk, blocks, steps)) return false;
    if (nk <= 128) return blocks >= (d_qk == 64 ? 256 : d_qk == 96 ? 192 : 224);
    return blocks >= (d_qk == 64 ? nk + nk / 5 : 160);
}

// ---- Variable-length calls, by the mean numbers of queries n and keys k per sequence (the host never sees the lengths).
// Shares are of the whole backward pass, kernel of the rule against the general one, over equal lengths of 8 ... 8192 and
// mixed ones, 4096 ... 65 536 tokens, H = 4/4 ... 16/16.

// Forward with 64 queries per wave (256-row blocks, one per CU) against the 128-row kernel (two per CU), for calls that do not
// take the decode kernel; nsplit = parts of the keys.  What decides is the length of a query's loop in a part, `loop`, beside
// the longer prologue and first two masked tiles of a lone block (us, 128-row -> this):
//   no mask  1000 keys 229 -> 229 ... 235, 1500 308 -> 293, 2000 397 -> 367, 6000 1081 -> 937 (d = 128; (192, 128) the same)
//   mask     self-attention of n: 1500 186 -> 212, 3000 316 -> 326, 4000 267 -> 260, 6000 557 -> 534; mixed 64 ... 8192 (1160 on
//            average) 612 -> 655; in one round of blocks the longest ends last (n = 4096, 256 blocks 83 -> 92)
//   chunk    512 queries x 32 heads against 8192 in 4 parts 79 -> 74, 16 384 140 -> 125, 32 768 270 -> 231; x 16 heads against 8192 in
//            8 parts of 1000 52 -> 53; 2 x 1024 x 16 against 3000 in 2 parts 58 -> 61
// and how the rows fill the blocks: 384 queries x 32 heads are 480 blocks of 128 rows, one round, but 320 of 256 in two: 112 -> 162.
inline bool fwd_one_wave_varlen(int d_qk, bool causal, int64_t B, int64_t Tq, int64_t Tk, int64_t H, int nsplit, bool uniform)
{
    if (d_qk != 128 && d_qk != 192) return false;
    const int64_t n = Tq / B, k = Tk / B, loop = (causal ? k - n / 2 : k) / nsplit;
    const int64_t large = (uniform ? B * ((n + 255) / 256) : (Tq + 255) / 256) * H * nsplit;
    const int64_t small = (uniform ? B * ((n + 127) / 128) : (Tq + 127) / 128) * H * nsplit;
    if (loop < (causal ? 1750 : 1200) || large <= (causal && k < 2 * n ? 256 : 128)) return false;
    return (large + 255) / 256 <= (small + 511) / 512;
}

// dQ with one wave per SIMD; half = 256-row blocks of queries x heads.
//   d = 128  64 queries per wave: half as many blocks as the 4-wave kernel, each with a CU to itself as there; with r rounds
//            of 256 blocks against s it takes 1.8 r to s.  n = 100 +11 ... +23 %, n = 512 -4 ... -11 %, n = 8192 -9 ... -20 %.
//            Under the mask a single round of short ragged sequences ends with its longest tile (5 x 800 +13 %), one of equal
//            lengths, whose 128-row blocks pair a long with a short tile per CU, at any length (2 x 1500 ... 6000 x 8 ... 16 heads
//            +5 ... +15 %; beyond one round -1 ... -12 %).
//   d = 64   the 4-wave kernel has two blocks per CU: n = 1024 +11 ... +26 % (mask), n = 2048 +5, n = 4096 -1, n = 8192 -5 %;
//            without the mask n = 800 +7, n = 2048 -3, n = 8192 -6 %.
//   (192, 128) and 256, 32 queries per wave, 128-row blocks as in the general kernel: n = 64 and less +5 ... +15 % (a tile
//            mostly empty costs the longer prologue), (192, 128) n = 512 without and 1024 with the mask -2 %, 256 from n = 100
//            or k = 1000 -2 ... -17 %.
inline bool dq_one_wave_varlen(int d_qk, bool causal, int64_t n, int64_t k, int64_t half, bool equal)
{
    const int64_t r = (half + 255) / 256, s = (2 * half + 255) / 256;
    if (d_qk == 128) return n >= 512 && 9 * r <= 5 * s && (!causal || half > 256 || (!equal && n >= 1500));
    if (d_qk == 64) return n >= (causal ? 4096 : 2048) && half >= 512;
    if (d_qk == 192) return n >= (causal ? 1024 : 512);
    return d_qk == 256 && (n > 64 || k > 64);
}

// dK/dV with one wave per SIMD (the same bits as the general kernels).
//   d = 128  n = k <= 32 +14 ... +17 %, 64 +3 ... +12, 100 -6 ... -12, 1000 -6 %; 16 queries against 1000 keys -2 %
//   (192, 128)  under the mask the same (n = k <= 64 +8 ... +13 %), without it -3 % at n = 8 and -50 % at n = 256
//   d = 256  two launches: under the mask n = k <= 64 +20 ... +32 %, 128 -8 ... +10, 64 against 4096 keys +20, 256 -1 ... -15;
//            without it n = 8 +6 ... 0, 32 -2 ... -19, 256 -33 ... -51 %
//   d = 64   256 keys per block and one block per CU against 128 and two: needs 512 blocks and long loops (n = 2048 +1 % with
//            and -5 % without the mask, n = 8192 -9 and -6 %); with four query heads per KV head +5 and +1 %
inline bool dkdv_one_wave_varlen(int d_qk, bool causal, int64_t n, int64_t k, int group, int64_t blocks_of_256_keys)
{
    const bool tiny = n <= 64 && k <= 64;
    if (d_qk == 128) return !tiny;
    if (d_qk == 192) return !tiny || !causal;
    if (d_qk == 256) return causal ? n > 128 : n > 16 || k > 16;
    return d_qk == 64 && n >= (causal ? 8192 : 2048) && group <= 2 && blocks_of_256_keys >= 512;
}

// ---- How the forward pass of a variable-length call runs.  Functions of the sizes alone (the host never sees
// the lengths, and the workspace is sized before the mask is known), so calls that share tables agree.
struct FwdRoute {
    bool decode;        // the kernel for few queries per sequence (attn_decode_kernel.inc)
    int nsub;           // its 32-row groups per (sequence, KV head)
    int nsplit;         // parts of the keys; 1: no partial results
};

inline FwdRoute fwd_route(int B, int Tq, int Tk, int H, int Hkv, int d_qk, int d_v, bool uniform)
{
    FwdRoute r{false, 1, 1};
    const int64_t G = H / Hkv, Nq = Tq / B, Nk = Tk / B;
    auto clamp = [](int64_t n, int64_t most) { return (int)(n < 1 || most < 1 ? 1 : n < most ? n : most); };
    auto root = [](int64_t n) { int64_t x = 0; while ((x + 1) * (x + 1) <= n) ++x; return x; };
    // Decode: a (sequence, KV head) is nsub groups of 32 rows there and G tiles of 128 rows in attn_fwd_kernel,
    // at about the same cost per group as per tile (B = 4, H = 32/8, Nk = 4096, d = 128: Nq = 16 31 us against
    // 44, Nq = 24 34 against 44, Nq = 32 45 against 45; G = 1: Nq = 64 46 against 41).  In a packed batch only
    // the totals are known; with no more queries than sequences it is the usual decode step, and a chunk among empty
    // slots has table entries for its queries (row_share in launch.h; 128 slots, one with 128 queries against 8192
    // keys, H = 32/8, d = 128: 65 us, 134 in 128-row tiles, 838 in the blocks of its own entry alone).  More queries
    // than sequences: the 128-row tiles.
    const int64_t nsub = ((uniform ? Nq : 1) * G + 31) / 32;
    const bool few_queries = uniform ? nsub == 1 || 4 * nsub <= 3 * G : Tq <= B;
    // ... but not against a few keys, for whose one to four tiles the merge of four waves costs as much as the work.  With
    // one head per KV head the 128-row kernel has no more blocks (B H = 4096, us, 128-row -> decode: d = 64 Nk = 64 22 -> 34,
    // 256 47 -> 56, 512 105 -> 109; d = 128 Nk = 64 36 -> 41, 320 126 -> 122; d = 256 Nk = 128 159 -> 164; (192, 128) Nk = 64
    // 52 -> 50); with more, where they all fit (B H <= 256, Nk <= 128: 4.1 -> 5.2, 5.0 -> 5.7, 7.1 -> 8.1 at 64, 128, 256).
    // (Packed lengths are uneven: 128 sequences of 16 ... 1024 keys, 235 on average, d = 64: 36 -> 35; empty slots have
    // no queries.)
    const int64_t keys = uniform ? Nk : Tk / Tq;
    const bool few_keys = (G == 1 && d_qk != 192 && keys <= (uniform && d_qk == 64 ? 256 : 128)) ||
                          (uniform && (int64_t)B * H <= 256 && Nk <= (d_qk == 192 ? 64 : 128));
    if (few_queries && !few_keys) {
        r.decode = true;
        r.nsub = (int)nsub;
        const int64_t items = (int64_t)B * Hkv * nsub, steps = (Nk + 127) / 128;
        if (items > 0xffffff) return r;
        if (!uniform) {
            // uneven lengths, longest first: four blocks per CU even out (48 sequences of 67 ... 7696 keys, 384
            // items: 91, 72, 63, 65 us for 1 ... 4 parts), of at least three steps of 128 keys on average; no more
            // than bring a sequence to 128 blocks by itself (one of 32 k keys, Hkv = 8: 33 us in 16 parts, 42 in 86)
            const int64_t even = (1023 + items) / items, alone = (127 + Hkv * nsub) / (Hkv * nsub);
            r.nsplit = clamp(even < alone ? even : alone, (steps + 2) / 3);
        } else if (items < 128) {
            // 128 blocks reach the memory's rate.  Parts of two steps and more (d = 64: three, 256: one), from six, for a part costs its
            // first loads and the merge (us, parts of four steps at least -> these: 4 x 1000 keys, Hkv = 8, d = 128 11.1 -> 9.7, 1 x 1000
            // 11.0 -> 9.7, 2 x 1316, Hkv = 2, d = 96 11.4 -> 9.4, 2 x 1100, d = 64 11.6 -> 10.5, 2 x 1000, d = 256 16.1 -> 11.6; 4 x 600, Hkv = 16,
            // d = 64 7.8 whole, 9.2 in two; B = 1, Hkv = 8, 32 k keys: 203 us in one part, 61 in 4, 40 in 8, 35 in 16, 40 in 32)
            // A part's loop shrinks as the merge's grows: the best number grows with the root of the keys (us, one KV head, parts of two steps at
            // least -> at most these: d = 128 32 k keys 24.2 in 128 -> 16.9 in 32, 21.0 in 16, 8 k 12.4 in 32, 12.0 in 16, 14.2 in 8; d = 64 32 k 19.5 in
            // 85, 16.2 in 32, 20.0 in 16; (192, 128) 32 k 25.4 in 128, 19.3 in 48, 19.5 in 32; d = 256 32 k 28.7 in 128, 22.6 in 64, 24.9 in 32, 8 k
            // 17.8 in 64, 15.5 in 32, 16.6 in 16)
            const int64_t least = d_qk == 64 ? 3 : d_qk > 192 ? 1 : 2, grows = root((d_qk > 192 ? 16 : d_qk == 192 ? 8 : d_qk == 64 ? 5 : 6) * steps);
            const int64_t most = d_qk > 192 && grows < 32 ? 32 : grows;
            const int64_t parts = steps / least <= most ? steps / least : (steps - 1) / ((steps - 1) / most + 1) + 1;      // (whole steps: none empty)
            r.nsplit = clamp((127 + items) / items, steps >= (d_qk > 192 ? 3 : 6) ? parts : 1);
            // (two parts of few steps: 64 ... 112 items, 6 and 7 steps d = 96, 128, 192 1.00 ... 1.18 of one part, d = 256 3 ... 7 steps 0.98 ... 1.15;
            // d = 64, 2 ... 112 items 0.99 ... 1.07; three and more 0.68 ... 1.01, from 8 steps 0.71 ... 0.97)
            if (r.nsplit == 2 && steps < 8) r.nsplit = 1;
        } else if (items > 256 && items < 1024) {
            // A last round of 256 that leaves CUs idle, in three parts per sequence, where the keys are long enough and
            // the round empty enough to pay for the partial results (three parts against one, 264 ... 320 / 352, 384 /
            // 448 ... 512 items: d = 128, Nk = 1000 0.97 ... 1.06 / 1.10 / 1.09, 2000 0.84 ... 0.91 / 0.98 / 1.07, 4000
            // 0.78 ... 0.88 / 0.95 / 1.04; d = 256, Nk = 1000 0.91 ... 0.97 / 1.05 / 1.12; d = 64, Nk = 2000 0.87 ... 0.97 /
            // 1.04 / 1.02, 4000 0.73 ... 0.84 / 0.87 / 0.98)
            const int64_t last = items % 256, elems = Nk * (d_qk + d_v);
            const bool pays = d_qk == 64 ? elems >= 250000 : elems >= 500000 && last <= (elems >= 1000000 ? 128 : 64);
            if (last != 0 && pays) r.nsplit = 3;
        }
    } else if (Tk > Tq) {
        // (self-attention is never divided: on whole tiles its bits are those of the fixed-length call where both run the
        // 128-row kernel)
        // Fewer blocks than the chip holds (two per CU, one at d = 256): divide the key loops, for the partial results travel
        // through memory in fp32: into parts of at least 4 tiles of 64 keys, from 12, while the blocks have a CU each, of at
        // least 16 where two share one (us, whole -> parts: 512 queries of 32 heads against 8 k keys 155 -> 92 in 2, 86 in 4, 95 in 8; 59 of 16
        // against 1687, B = 3, d = 96 25.9 -> 15.7 in 5; 34 of 16 against 1359, B = 2, d = 256 49.7 -> 23.9 in 5; 100 of 32 against 2000
        // 36.6 -> 20; 128 of 16 against 2000, B = 2 37.7 -> 19.2 in 7; 1000 of 8 against 4000 36.7 in 3, 32.2 in 4, 33.4 in 8; 600 of 8 against
        // 1200, d = 64 16.8 -> 14.1 in 3; 128 queries of 32 heads against 600 keys 15.7 whole, 16.5 in 2; 500 of 16 against 700 16.9 and 19.4;
        // two per CU: 200 of 16 against 3000, B = 4 55.6 whole, 41.4 in 2, 44.6 in 4, 100 of 32 against 4000 65, 53 in 3, 47 in 4; 2048 of 16 heads
        // against themselves, whose loops are half as long: 42 whole, 49 in 2)
        const int64_t blocks = (uniform ? (int64_t)B * ((Nq + 127) / 128) : (int64_t)Tq / 128 + B) * H;
        // The parts of blocks that are alone are no more than pay for their merge, as above (us, 31 ... 127 parts of four tiles -> at most these; parts
        // of 16 tiles: 64 queries of one head, d = 64 32 k keys 27.8 in 127, 20.8 in 48, 22.7 in 31, 8 k 14.2 in 31, 13.3 in 24, 20.5 in 7; d = 128
        // 32 k 30.4 in 127, 25.4 in 48, 28.8 in 31; d = 256 32 k 39.4 in 127, 34.8 in 64, 49.0 in 31; 300 of 4, d = 64 8 k 17.2 in 21, 16.7 in 16)
        const int64_t tiles = (Nk - Nq / 2) / 64, most = root((d_qk > 128 ? 9 : 4) * tiles);
        // (a packed batch may hold any lengths: parts of 16 tiles of the mean, and the workspace that this needs)
        const int alone = clamp(256 / blocks, uniform && tiles >= 12 ? tiles / 4 < most ? tiles / 4 : most : 1), shared = clamp((d_qk > 192 ? 256 : 512) / blocks, tiles / 16);
        r.nsplit = alone > shared ? alone : shared;
    }
    return r;
}

// The parts that a decode step of equal lengths launches, of nsplit: a part is whole steps of 128 keys, so that the last ones may be left without
// any (2000 keys in 5: 4 parts of 4 steps).  At d = 64 these are not launched (2048 keys, one head 9.4 us with the empty part, 9.0 without; 3513 keys x 5
// in 9 1.07 of 7).  At larger head dims they cost less than how another number falls on the chip's eight dies (9242 keys, Hkv = 8, 15 parts
// against 16 with one empty: d = 96 14.0 and 12.9, d = 128 14.3 and 15.6; 6500 keys, d = 96, 13 of 16 12.4 and 11.8).
inline int parts_with_keys(const FwdRoute& r, bool uniform, int d_qk, int nk, int nsplit)
{
    if (!uniform || !r.decode || d_qk != 64 || nsplit <= 1) return nsplit;
    const int steps = nk / 128 + (nk % 128 != 0), per = (steps - 1) / nsplit + 1;
    return (steps - 1) / per + 1;
}

// Blocks of the merge kernel that share the rows of a tile, in turns of 1024 / d_v rows per block.  On the decode route a
// packed tile holds one query as a rule; the 128-row kernel's tiles hold up to 128 (shares past a short one's rows end at
// once: at most 4096 blocks, for only calls of few tiles are divided).  512 packed queries, H = 32/8, 8192 keys, three
// parts: 91 us, 141 undivided, and 133 with the 40 blocks of 64 turns each that one query per tile would ask for.
inline int merge_shares(const FwdRoute& r, bool uniform, int nq, int group, int d_v)
{
    const int rows = (uniform ? (nq < 128 ? nq : 128) : r.decode ? 1 : 128) * group, per = 1024 / d_v;
    return (rows + per - 1) / per;
}

}  // namespace attn
