// Host-side argument bundles handed from the C ABI to the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdlib.h>
#include <tuple>
#include "dispatch.h"

namespace attn {

// Element strides of one tensor in the variable-length kernels: the address of (token t, head h) of
// sequence s is  base + t * row + s * batch + h * head  (+ the position inside the head dim), t
// being the token's index in the packed batch.  Packed tensors have batch = 0; a [B, N, ...]
// tensor whose batch stride is not N rows passes batch = (batch stride) - N * row.
struct Stride3 {
    long long batch, row, head;
};
struct VarlenStrides {
    Stride3 q, k, v, o, d_o, dq, dk, dv;
    long long lse_batch, lse_head;      // lse index = t + s * lse_batch + h * lse_head
    // equal-length batches (the strided calls): every sequence has nq queries and nk keys, and a kernel
    // computes its tile-table entry (placed_entry) instead of reading one; 0: the tables say
    int nq, nk;
};

// Mark of a used entry of the tile tables.  Not 1: a workspace that was never planned, or whose
// tables were overwritten, then holds no entry that a kernel would act on.
constexpr int kPlanUsed = 0x5A17AB1E;
// Mark of an entry behind the used ones that takes a share of another tile's rows in the decode and merge kernels (see
// row_share); the other kernels pass over it like over an unused one.
constexpr int kPlanHelp = 0x5A17AB1F;

// Entry e of the table of query tiles: seq = {first query row, query length, first key row, key length} of the sequence,
// til = {tile of 128 rows inside it, kPlanUsed, sequence, helpers}; a sequence's tiles are listed last to first.
// Equal-length batches need no table: the entry follows from e, which spares the strided calls the two
// boundary kernels and the plan kernel (three launches in a row, 10 us of a call).
__device__ __forceinline__ void query_tile_entry(const int4* __restrict__ plan, int e, const VarlenStrides& st, int4& seq, int4& til)
{
    if (st.nq > 0) {
        const int nt = (st.nq + 127) / 128;
        const int b = e / nt;
        seq = make_int4(b * st.nq, st.nq, b * st.nk, st.nk);
        til = make_int4(nt - 1 - (e - b * nt), kPlanUsed, b, 0);
    } else {
        seq = plan[2 * e];
        til = plan[2 * e + 1];
    }
}

// (head, tile) of a place in a launch over equal lengths (the functions of dispatch.h in scalar registers).
template <bool CAUSAL>
__device__ __forceinline__ HeadTile uniform_head_tile(const TileOrder& order, Place place, int tiles)
{
    HeadTile ht;
    if constexpr (CAUSAL) {
        TileOrder o = order;
        asm volatile("" : "+s"(o.group), "+s"(o.own_group), "+s"(o.unit), "+s"(o.own));     // loaded at once, not each behind its branch
        ht = head_tile(o, place, tiles);
    } else {
        ht = head_tile_in_shares(order, place, tiles);
    }
    return {__builtin_amdgcn_readfirstlane(ht.head), __builtin_amdgcn_readfirstlane(ht.tile)};
}
// (head, entry) of a place in a launch over a table.
__device__ __forceinline__ HeadTile uniform_head_entry(const TileOrder& order, Place place, int entries)
{
    const HeadTile ht = head_tile_in_units(order, place, entries);
    return {__builtin_amdgcn_readfirstlane(ht.head), __builtin_amdgcn_readfirstlane(ht.tile)};
}

// The table entry and the head of a place in the launch's order (query_order, key_order); where equal lengths need no table,
// it follows from the place, for blocks of two tiles that of the first of them.
template <bool QUERY_SIDE, bool CAUSAL, int ROWS = 128>
__device__ __forceinline__ void placed_entry(const int4* __restrict__ plan, const TileOrder& order, Place place, int max_tiles, int heads,
                                             const VarlenStrides& st, int& head, int4& seq, int4& til)
{
    if (st.nq > 0) {
        const int n = QUERY_SIDE ? st.nq : st.nk, nt = (n + ROWS - 1) / ROWS;
        const HeadTile ht = uniform_head_tile<CAUSAL>(order, place, nt);
        const int b = ht.head / heads;
        head = ht.head - b * heads;
        seq = make_int4(b * st.nq, st.nq, b * st.nk, st.nk);
        // (query tiles: the last has the longest loop under the mask; key tiles, which the tables list backwards: the first)
        til = make_int4(QUERY_SIDE ? (ROWS / 128) * (nt - 1 - ht.tile) : (n + 127) / 128 - 1 - (ROWS / 128) * ht.tile, kPlanUsed, b, 0);
    } else {
        const HeadTile ht = uniform_head_entry(order, place, max_tiles);
        head = ht.head;
        seq = plan[2 * ht.tile];
        til = plan[2 * ht.tile + 1];
    }
}

// The rows of a tile in units, for the decode and merge kernels: n blocks per entry, block i of entry e takes units `unit`,
// `unit` + `step`, ...  n units hold the rows of one query.  In a packed batch with no more queries than sequences a tile
// usually is one query; where one holds more (a prompt chunk among empty slots), each further query has an entry of its
// own behind the used ones (kPlanHelp: {tile's entry, query within it}; there is room, since queries <= sequences), so
// that every block takes one unit and the chunk is spread over the chip.  til.w != 0: the tile has such helpers; 0 (and
// equal lengths, whose n covers the whole tile): the entry's blocks take all units.
__device__ __forceinline__ bool row_share(const int4* __restrict__ plan, int e, int max_tiles, const VarlenStrides& st, int T,
                                          int i, int n, int4& seq, int4& til, int& unit, int& step)
{
    constexpr int one_turn = 1 << 24;
    query_tile_entry(plan, e, st, seq, til);
    unit = i;
    step = til.w != 0 ? one_turn : n;
    if (til.y == kPlanHelp) {
        const int of = seq.x, query = seq.y;
        if (of < 0 || of >= max_tiles || query < 1 || query > 127) return false;
        seq = plan[2 * of];
        til = plan[2 * of + 1];
        unit += query * n;
        step = one_turn;
    }
    return til.y == kPlanUsed && seq.x >= 0 && seq.y >= 0 && seq.x + seq.y <= T;
}

// The same for a packed batch of at most 64 sequences with no more queries than sequences, without a table: every wave finds
// entry e from the boundaries, a sequence per lane.  All tiles are first ones (a sequence has at most 64 queries).  The entries
// are those that varlen_plan_kernel makes of such a batch, sequences with the most keys first (ties by index), and are
// returned as the table holds them (rows, tile).  A table kernel before a decode step of 48 sequences is 5 us and a launch.
__device__ __forceinline__ bool row_share_of_few(const int* __restrict__ cu_q, const int* __restrict__ cu_k, int B, int Tq, int Tk,
                                                 int e, int max_tiles, int i, int n, int4& seq, int4& til, int& unit, int& step,
                                                 int4& rows, int4& tile)
{
    constexpr int one_turn = 1 << 24;
    const int l = threadIdx.x & 63, b = min(l, B - 1);
    const int qs = cu_q[b], ql = cu_q[b + 1] - qs, ks = cu_k[b], kl = cu_k[b + 1] - ks;
    const bool inside = l < B && qs >= 0 && ql > 0 && qs <= Tq - ql && ks >= 0 && kl > 0 && ks <= Tk - kl;
    const int key = inside ? kl : 0, more = inside ? ql - 1 : 0;        // keys; queries beside the first
    const uint64_t used = __ballot(inside), chunks = __ballot(more > 0);
    // (boundaries that overlap may list more queries than there is room for)
    auto helps = [&](int before) { return more > 0 && __popcll(used) + before + more <= max_tiles; };
    const int total = __popcll(used), h = e - total;
    uint64_t mine = 0;
    int before = 0;
    auto below = [&](uint64_t lanes) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0)); };
    if (h < 0) {
        // the (e + 1)-th most keys, bit by bit (ranks of all lanes, one lane after the other: 3 us more per step of 48)
        int t = 0;
        for (int bit = 31 - __builtin_clz(Tk); bit >= 0; --bit)
            if (__popcll(__ballot(key >= (t | 1 << bit))) > e) t |= 1 << bit;
        const uint64_t equal = __ballot(key == t);
        const int place = e - __popcll(__ballot(key > t));              // among those of as many keys
        mine = __ballot(key == t && below(equal) == place);
    } else if (chunks) {
        for (uint64_t left = chunks; left; left &= left - 1) {
            const int m = __builtin_ctzll(left), mm = __builtin_amdgcn_readlane(more, m);
            before += m < l ? mm : 0;
        }
        mine = __ballot(helps(before) && before <= h && h < before + more);
    }
    rows = tile = make_int4(0, 0, 0, 0);
    if (!mine) return false;
    const int s = __builtin_ctzll(mine);
    auto of = [&](int x) { return __builtin_amdgcn_readlane(x, s); };
    seq = make_int4(of(qs), of(ql), of(ks), of(kl));
    if (h < 0 && of(more) > 0)
        for (uint64_t left = chunks & ((1ull << s) - 1); left; left &= left - 1) before += __builtin_amdgcn_readlane(more, __builtin_ctzll(left));
    til = make_int4(0, kPlanUsed, s, of(helps(before)));
    unit = i;
    step = til.w != 0 ? one_turn : n;
    rows = seq;
    tile = til;
    if (h >= 0) {
        const int query = h - of(before) + 1;
        rows = make_int4(__popcll(__ballot(key > seq.w)) + __popcll(__ballot(key == seq.w) & ((1ull << s) - 1)), query, 0, 0);
        tile = make_int4(0, kPlanHelp, 0, 0);
        unit += query * n;
    }
    return true;
}

struct FwdArgs {
    const void *q, *k, *v;
    void* o;
    float* lse;
    int B, H, Hkv, N, d_qk, d_v;
    float scale;
    int causal;
    void* stream;
    // variable-length mode (max_tiles > 0): N unused; plan = table of query tiles (unread if st.nq > 0), max_tiles its size
    // (an upper bound on the number of 128-row query tiles), T and Tk = total query and key rows
    const void* plan = nullptr;
    int T = 0, max_tiles = 0, Tk = 0;
    VarlenStrides st = {};   // variable-length mode: q, k, v, o and lse strides
    bool f16 = false;   // 16-bit storage type of q, k, v, o: bf16 (default) or IEEE fp16
    // variable-length mode: keys of a sequence divided over nsplit blocks whose unnormalised results go to
    // part_o [nsplit][T][H][d_v] and part_ml [nsplit][T][H] {reference maximum, row sum} (nsplit > 1)
    int nsplit = 1;
    float *part_o = nullptr, *part_ml = nullptr;
    int nsub = 1;       // decode kernel: blocks per table entry that share the 32-row groups of a tile (row_share)
    int nshare = 1;     // merge kernel: blocks per table entry that share the rows of a tile
    const int *cu_q = nullptr, *cu_k = nullptr;     // decode kernel: boundaries to make the table of (row_share_of_few)
};

struct BwdArgs {
    const void *q, *k, *v, *o, *d_o;
    const float* lse;
    void *dq, *dk, *dv;
    int B, H, Hkv, N, d_qk, d_v;
    float scale;
    int causal;
    // workspace carved up by the API: -D = -rowsum(dO o O) and the base-2 LSE
    float* D;
    float* lse2;
    void* stream;
    int phases;   // bit mask: 1 prepare, 2 dK/dV kernel, 4 dQ kernel
    const void* plan = nullptr;   // variable-length mode (max_tiles > 0), as in FwdArgs: query-tile table (dQ kernel)
    int T = 0, max_tiles = 0;
    const void* plan_k = nullptr; // key-tile table (dK/dV kernels), its size, and the total of key rows
    int max_tiles_k = 0, Tk = 0;
    VarlenStrides st = {};        // variable-length mode: strides of every tensor and of lse
    int rows_per_batch = 0;       // variable-length mode, prepare kernel: tokens per sequence when the
                                  // tensors have a batch stride (equal lengths), 0 for packed tensors
    bool f16 = false;             // as in FwdArgs
};

// Launch through hipLaunchKernel so that the status returned belongs to THIS launch (the
// sticky hipGetLastError slot may hold an unrelated earlier error of the host program).
template <typename... KArgs, typename... Args>
inline hipError_t launch_kernel(void (*kern)(KArgs...), dim3 grid, dim3 block, size_t smem, void* stream,
                                Args... args)
{
    std::tuple<KArgs...> vals{static_cast<KArgs>(args)...};
    void* ptrs[sizeof...(KArgs)];
    int n = 0;
    std::apply([&](auto&... v) { ((ptrs[n++] = (void*)&v), ...); }, vals);
    return hipLaunchKernel((const void*)kern, grid, block, ptrs, smem, (hipStream_t)stream);
}

// Raises a kernel's dynamic-LDS limit to `smem` bytes on the current device.  The attribute
// belongs to the (kernel, device) pair, so the "already done" note is kept per device; a race
// between two host threads only repeats the idempotent call.
struct LdsOptIn {
    bool done[64] = {};
    template <typename K>
    bool allow(K kern, int smem)
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return false;
        if (dev >= 0 && dev < 64 && done[dev]) return true;
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
            return false;
        if (dev >= 0 && dev < 64) done[dev] = true;
        return true;
    }
};

// 0 on success, -2 unsupported head dims, -3 launch failure.
int launch_fwd(const FwdArgs& a);
int launch_bwd(const BwdArgs& a);
// The 64-queries-per-wave forward kernel (head dims 128, 64 or (192, 128), fixed length, N % 256 = 0; or 128 or (192, 128) in
// variable-length mode with row strides of at least a row).
int launch_fwd_q64(const FwdArgs& a);
// The decode kernel (variable-length mode, every head dim): few queries per sequence; and the merge of the
// partial results of a pass with nsplit > 1.
int launch_decode(const FwdArgs& a);
int launch_combine(const FwdArgs& a);
// The dQ kernel with 64 queries per wave (d_qk = d_v = 128 or 64; fixed length N % 256 = 0, or variable-length
// mode with row strides of at least a row); it also leaves -D and the base-2 LSE of every row in the workspace.
// Which calls these launchers get: dispatch.h.
int launch_bwd_dq_q64(const BwdArgs& a);
// The dK/dV kernel with one wave per SIMD and 32-query tiles (head dims 128, (192, 128) and 256, there as a dV and a
// dK launch: N % 128 = 0; 64: N % 256 = 0; or variable-length mode as above; with or without the causal mask); -D and
// the base-2 LSE must be in the workspace.
int launch_bwd_dkdv_t32(const BwdArgs& a);
// The dQ kernel with one wave per SIMD and 32 queries per wave (head dims (192, 128) and 256; fixed length
// N % 128 = 0, or variable-length mode as above); it also leaves -D and the base-2 LSE of every row in the workspace.
int launch_bwd_dq_t32(const BwdArgs& a);
// dQ, dK and dV in one kernel, one block per (sequence, KV head) (d_qk = d_v = 64 up to 512 keys, 96 or 128 up to 256; equal lengths, in
// variable-length mode with row strides of at least a row); what it writes: dQ with phases & 4, dK and dV with phases & 2.
int launch_bwd_short(const BwdArgs& a);
// The kernels with one wave per SIMD by element type (bf16 in attn::, fp16 in attn::f16k::) and mode: one translation unit each.
int run_bwd_dq_q64(const BwdArgs& a);
int run_bwd_dq_t32(const BwdArgs& a);
int run_bwd_dkdv_t32(const BwdArgs& a);
int run_bwd_dq_q64_varlen(const BwdArgs& a);
int run_bwd_dq_t32_varlen(const BwdArgs& a);
int run_bwd_dkdv_t32_varlen(const BwdArgs& a);
namespace f16k {
int run_bwd_dq_q64(const BwdArgs& a);
int run_bwd_dq_t32(const BwdArgs& a);
int run_bwd_dkdv_t32(const BwdArgs& a);
int run_bwd_dq_q64_varlen(const BwdArgs& a);
int run_bwd_dq_t32_varlen(const BwdArgs& a);
int run_bwd_dkdv_t32_varlen(const BwdArgs& a);
}  // namespace f16k
// Fills the two plan tables of the variable-length entry points on the device: 0 or -3.
int launch_varlen_plan(const int* cu_q, const int* cu_k, int B, int Tq, int Tk, void* plan_q, int max_tiles_q,
                       void* plan_k, int max_tiles_k, void* stream);

}  // namespace attn
