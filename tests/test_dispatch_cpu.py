"""CPU checks of csrc/dispatch.h, built alone with the host compiler: the order in which blocks take table entries, and the
rules that choose kernels."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_05451_amd", "csrc")

SHIM = r"""
#include "dispatch.h"
using namespace attn;
extern "C" {
int t_section_order(int block, int total) { return section_order(block, total); }
int t_order(int block, int heads, int tiles, int share, long long bytes, int causal, int half_empty)
{
    const TileOrder o = causal ? causal_order(heads, tiles, share, bytes) : tile_order(heads, tiles);
    const int total = heads * tiles;
    const HeadTile t = head_tile(o, half_empty ? block_place_alternate(o, block, total) : block_place(o, block), tiles);
    return t.head * tiles + t.tile;
}
// What block `block` of a launch over the query (key) tiles of an equal-length batch does: head * 2^16 + 128-row tile, counted
// from the longest loop; -1 past the launch.
struct Args { int B, H, Hkv, N, d_qk, d_v, causal, max_tiles, max_tiles_k; struct { int nq, nk; } st; };
int t_equal(int block, int keys, int B, int H, int Hkv, int nq, int nk, int d, int causal, int rows)
{
    const Args a{B, H, Hkv, 0, d, d, causal, B * ((nq + 127) / 128), B * ((nk + 127) / 128), {nq, nk}};
    const int total = keys ? key_blocks(a, rows) : query_blocks(a, rows);
    if (block >= total) return -1;
    const TileOrder o = keys ? key_order(a, rows) : query_order(a, rows);
    const HeadTile t = head_tile(o, entry_place(o, rows, true, block, total), keys ? tiles_of_key_launch(a, rows) : tiles_of_query_launch(a, rows));
    return t.head * 65536 + t.tile * (rows / 128);
}
// Whether the short forms of head_tile give what it gives on the orders that they are for.
int t_same(int heads, int tiles)
{
    const TileOrder s = share_order(heads, tiles), u = tile_order(heads, tiles);
    for (int b = 0; b < heads * tiles; ++b) {
        const HeadTile x = head_tile(s, block_place(s, b), tiles), y = head_tile_in_shares(s, block_place(s, b), tiles);
        const HeadTile z = head_tile(u, block_place(u, b), tiles), w = head_tile_in_units(u, block_place(u, b), tiles);
        if (x.head != y.head || x.tile != y.tile || z.head != w.head || z.tile != w.tile) return 0;
    }
    return 1;
}
int t_fwd_varlen(int d, int causal, int B, int Tq, int Tk, int H, int Hkv, int uniform)
{
    const FwdRoute r = fwd_route(B, Tq, Tk, H, Hkv, d, 128, uniform);
    return !r.decode && fwd_one_wave_varlen(d, causal, B, Tq, Tk, H, r.nsplit, uniform);
}
int t_turns(int heads, int tiles, int causal)
{
    return takes_turns(causal ? causal_order(heads, tiles, 1, 1) : tile_order(heads, tiles), tiles, (long long)heads * tiles, causal);
}
int t_fwd(int d, int causal, int N, long long b) { return fwd_one_wave(d, causal, N, b); }
int t_dq(int d, int causal, int N, long long b) { return dq_one_wave(d, causal, N, b); }
int t_dkdv64(int d, int causal, int N, long long b) { return dkdv64_one_wave(causal, N, b); }
int t_dq256(int causal, int N, long long heads) { return dq256_one_wave(causal, N, heads); }
int t_dkdv256(int N, long long heads) { return dkdv256_one_wave(N, heads); }
int t_lean(int d, int causal, long long blocks, long long loop) { return lean_blocks(d, causal, blocks, loop); }
int t_lean_dq(int d, int causal, long long blocks, long long nq, long long nk) { return lean_dq_blocks(d, causal, blocks, nq, nk, false); }
int t_lean_strided(int causal, long long blocks, long long loop) { return lean_blocks(64, causal, blocks, loop, true); }
int t_tiles(int equal, int max_tiles, int T, int B) { return (int)likely_tiles(equal, max_tiles, T, B); }
int t_short(int d, int causal, int nq, int nk, int B, int H, int Hkv) { return bwd_short(d, d, causal, nq, nk, B, H, Hkv); }
int t_live(int uniform, int decode, int d, int nk, int nsplit) { return parts_with_keys(FwdRoute{decode != 0, 1, nsplit}, uniform, d, nk, nsplit); }
int t_route(int B, int Tq, int Tk, int H, int Hkv, int dqk, int dv, int uniform, int* nsplit)
{
    const FwdRoute r = fwd_route(B, Tq, Tk, H, Hkv, dqk, dv, uniform);
    *nsplit = r.nsplit;
    return r.decode;
}
int t_shares(int B, int Tq, int Tk, int H, int Hkv, int dqk, int dv, int uniform)
{
    return merge_shares(fwd_route(B, Tq, Tk, H, Hkv, dqk, dv, uniform), uniform, Tq / B, H / Hkv, dv);
}
int t_dq_varlen(int d, int causal, long long n, long long k, long long half) { return dq_one_wave_varlen(d, causal, n, k, half, false); }
int t_dkdv_varlen(int d, int causal, long long n, long long k, int group, long long blocks64)
{ return dkdv_one_wave_varlen(d, causal, n, k, group, blocks64); }
}
"""


@pytest.fixture(scope="module")
def D(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"),
                    "-o", str(d / "shim.so")], check=True)
    L = ctypes.CDLL(str(d / "shim.so"))
    q = ctypes.c_longlong
    L.t_order.argtypes = [ctypes.c_int] * 4 + [q] + [ctypes.c_int] * 2
    for f in (L.t_fwd, L.t_dq, L.t_dkdv64):
        f.argtypes = [ctypes.c_int] * 3 + [q]
    L.t_dq_varlen.argtypes = [ctypes.c_int] * 2 + [q] * 3
    L.t_dkdv_varlen.argtypes = [ctypes.c_int] * 2 + [q] * 2 + [ctypes.c_int, q]
    return L


@pytest.mark.parametrize("heads", [1, 2, 3, 4, 6, 8, 16, 32])
@pytest.mark.parametrize("lens", [[4096] * 16, [8192, 129, 700], [300] * 40, [257, 1025, 640, 64]])
def test_places_of_blocks_that_take_two_tiles(D, heads, lens):
    """Every place once; with a total that is dealt to the XCDs, every XCD has its share of the live places (those of a
    sequence's even tiles) and does not get them behind all of its empty ones."""
    max_tiles = sum(lens) // 128 + len(lens)
    tiles = [t for n in lens for t in range((n + 127) // 128 - 1, -1, -1)]              # a table: last tile first
    live = np.array([t % 2 == 0 for t in tiles] + [False] * (max_tiles - len(tiles)))
    total = max_tiles * heads
    places = np.array([D.t_section_order(b, total) for b in range(total)])
    assert sorted(places) == list(range(total))
    if total % 8:
        return
    took = live[places % max_tiles]
    for xcd in range(8):
        mine = places[xcd::8]
        assert mine.min() == xcd * (total // 8) and mine.max() == (xcd + 1) * (total // 8) - 1       # one section
        want = live[mine % max_tiles].sum()
        assert took[xcd::8].sum() == want
        used = (mine % max_tiles < len(tiles)).sum()            # half of a section's used entries, and one per sequence
        assert used / 2 - 1 <= want <= used / 2 + len(lens) * (1 + heads // 8)


@pytest.mark.parametrize("heads", [1, 2, 3, 4, 5, 8, 12, 16, 20, 33, 36, 63, 96, 98, 100, 136, 248])
@pytest.mark.parametrize("tiles", [1, 2, 3, 8, 16, 31, 64])
@pytest.mark.parametrize("half_empty", [0, 1])
def test_order_of_blocks(D, heads, tiles, half_empty):
    """Every (head, tile) once, whatever the heads, tiles and group; without the mask an XCD with heads of its own takes them one
    after the other; under it no XCD gets much more work than another, and its blocks go from long to short within a group.
    Half empty: launches over tables, whose order is the same with and without the mask; an XCD's live places fall alike on
    the four positions modulo 4, and no XCD gets many fewer of them."""
    total = heads * tiles
    assert D.t_same(heads, tiles)
    for causal, share, nbytes in ((0, 1, 1), (1, 1, 1), (1, 1, 5 << 20), (1, 4, 5 << 20), (1, 1, 1 << 40)):
        at = np.array([D.t_order(b, heads, tiles, share, nbytes, causal, half_empty) for b in range(total)])
        assert sorted(at) == list(range(total)), (causal, share, nbytes)
        if total % 8:
            continue
        if half_empty:
            if not causal and tiles % 2 == 0:       # (a table's sequences of an even number of tiles: every second place is live)
                for xcd in range(8):
                    live = np.array([(at[b] % tiles) % 2 == 0 for b in range(xcd, total, 8)])
                    assert abs(live.sum() - total / 16) <= 1
                    by_position = [live[i::4].sum() for i in range(4)]
                    assert max(by_position) - min(by_position) <= 2
            continue
        for xcd in range(8):
            mine = at[xcd::8]
            if not causal and heads % 8 == 0:
                assert (mine == np.arange(xcd * total // 8, (xcd + 1) * total // 8)).all()
            if causal:
                work = tiles - mine % tiles                         # tile 0 has the longest loop
                # (at most one block per CU ends with its longest tile however the work is shared)
                assert total <= 256 or abs(work.sum() - heads * tiles * (tiles + 1) / 16) <= tiles * max(1, heads // 8) / 2
                falls = (np.diff(mine % tiles) < 0).sum() + 1       # a new group starts
                unit = max(1, heads // 8) if heads % 8 == 0 else 0
                if unit and nbytes == 1:
                    assert falls == max(1, unit // 8) or tiles == 1
                if unit and nbytes == 1 << 40:
                    assert falls == unit or tiles == 1


@pytest.mark.parametrize("B,H,Hkv,N,d", [(2, 16, 16, 4096, 128), (1, 32, 32, 8192, 128), (2, 8, 8, 4096, 128), (2, 16, 16, 4000, 128),
                                         (8, 16, 16, 1000, 128), (1, 12, 4, 2300, 128), (3, 5, 5, 513, 64), (2, 16, 16, 8192, 64)])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("keys", [0, 1])
def test_equal_lengths_in_blocks_of_256_rows(D, B, H, Hkv, N, d, causal, keys):
    """Equal lengths, kernels that take two 128-row tiles: every pair of tiles once, no block without one (empty blocks that
    alternate with live ones leave half of the shader engines idle), and under the mask an XCD's blocks from long to short within a
    group of heads."""
    tiles, heads = (N + 255) // 256, B * (Hkv if keys else H)
    at = [D.t_equal(b, keys, B, H, Hkv, N, N, d, causal, 256) for b in range(heads * tiles + 1)]
    assert at.pop() == -1
    assert sorted(at) == [h * 65536 + 2 * t for h in range(heads) for t in range(tiles)]
    if causal and len(at) % 8 == 0:
        for xcd in range(8):
            mine = np.array(at[xcd::8]) % 65536 // 2
            falls = np.flatnonzero(np.diff(mine) < 0) + 1           # a new group starts, with its longest tile
            assert (mine[falls] == mine[0]).all() and len(falls) + 1 <= max(1, heads // 8)


@pytest.mark.parametrize("B,H,N,causal,rows", [(1, 31, 1024, 0, 128), (1, 15, 4096, 0, 128), (3, 5, 2000, 0, 128), (1, 13, 2048, 1, 128),
                                               (1, 12, 2048, 1, 128), (1, 7, 8192, 0, 256), (2, 10, 4096, 0, 128), (1, 31, 2048, 1, 256)])
@pytest.mark.parametrize("keys", [0, 1])
def test_shares_of_equal_work(D, B, H, N, causal, rows, keys):
    """Equal tiles, or no more blocks than CUs: an XCD reads the rows of no more heads than its share of the tiles spans, whatever
    the number of heads."""
    tiles = (N + rows - 1) // rows
    total = B * H * tiles
    assert total % 8 == 0 and (not causal or total <= 256)
    at = np.array([D.t_equal(b, keys, B, H, H, N, N, 128, causal, rows) for b in range(total)])
    assert len(set(at)) == total
    for xcd in range(8):
        assert len(set(at[xcd::8] // 65536)) <= (total // 8 - 1) // tiles + 2


@pytest.mark.parametrize("heads,tiles", [(63, 8), (45, 8), (100, 4), (202, 4), (47, 16), (33, 32), (255, 8), (17, 32), (25, 16)])
def test_heads_of_its_own_before_shared_ones(D, heads, tiles):
    """Under the mask, many heads that do not divide: an XCD reads the rows of its own eighth of the heads, rounded down, and of the few
    that are left over, and within either its blocks go from long to short."""
    total = heads * tiles
    for xcd in range(8):
        at = np.array([D.t_order(b, heads, tiles, 1, 1, 1, 0) for b in range(xcd, total, 8)])
        assert len(set(at // tiles)) <= heads // 8 + heads % 8
        assert (np.diff(at % tiles) < 0).sum() <= 1 + max(1, heads // 8 // 8)


def test_turns(D):
    """Two turns and more; under the mask whole pairs of them, of heads that an XCD has to itself."""
    import test_gpu_few_blocks as S
    for causal, N, Hkv, _ in S.TURNS:
        assert D.t_turns(Hkv, N // 128, causal), (causal, N, Hkv)
    assert not D.t_turns(256, 1, 0) and not D.t_turns(4, 64, 1) and not D.t_turns(36, 17, 1) and not D.t_turns(84, 9, 1)
    assert not D.t_turns(32, 64, 1) and D.t_turns(32, 64, 0)
    for N, Hkv, _ in S.TURNS64:
        assert D.t_dkdv64(64, 0, N, Hkv * N // 256) and D.t_turns(Hkv, N // 256, 0), (N, Hkv)


# measured times of the kernels with one wave per SIMD over those of the 4-wave kernels: (pass, d, causal, N, 256-row blocks,
# ratio), both sides of every line of the rules; under the mask with the tiles of groups of heads taken together
MEASURED = [
    ("fwd", 128, 0, 8192, 128, 1.08), ("fwd", 128, 0, 2048, 136, 0.78), ("fwd", 128, 0, 1024, 256, 0.95), ("fwd", 128, 0, 1024, 264, 1.16),
    ("fwd", 128, 0, 2048, 416, 0.85), ("fwd", 64, 0, 1024, 160, 1.04), ("fwd", 64, 0, 2048, 256, 0.94), ("fwd", 64, 0, 8192, 320, 1.24),
    ("fwd", 64, 0, 8192, 448, 0.92), ("fwd", 64, 0, 4096, 576, 1.19), ("fwd", 64, 0, 4096, 480, 0.92),
    ("fwd", 64, 0, 6144, 960, 0.92), ("fwd", 64, 0, 7168, 896, 1.03), ("fwd", 64, 0, 3072, 960, 1.02), ("fwd", 128, 1, 1024, 136, 1.33),
    ("fwd", 128, 1, 2048, 160, 1.22), ("fwd", 128, 1, 3072, 192, 1.15), ("fwd", 128, 1, 4096, 256, 1.08), ("fwd", 128, 1, 8192, 256, 1.05),
    ("fwd", 128, 1, 4096, 320, 1.03), ("fwd", 128, 1, 4096, 384, 0.94), ("fwd", 128, 1, 4096, 448, 0.91), ("fwd", 128, 1, 3072, 576, 1.03),
    ("fwd", 128, 1, 6144, 384, 0.97), ("fwd", 128, 1, 8192, 512, 0.88), ("fwd", 192, 1, 2048, 256, 1.08), ("fwd", 192, 1, 3072, 240, 1.03),
    ("fwd", 192, 1, 4096, 192, 1.05), ("fwd", 192, 1, 4096, 208, 0.89), ("fwd", 192, 1, 7168, 168, 1.03), ("fwd", 192, 1, 7168, 224, 0.99),
    ("fwd", 192, 1, 8192, 192, 0.99), ("fwd", 192, 1, 3072, 576, 1.02), ("fwd", 192, 1, 4096, 384, 0.93), ("fwd", 192, 1, 6144, 288, 0.98),
    ("fwd", 64, 1, 4096, 448, 1.15), ("fwd", 64, 1, 8192, 384, 1.04), ("fwd", 64, 1, 8192, 448, 0.93), ("fwd", 64, 1, 8192, 640, 1.08),
    ("fwd", 64, 1, 12288, 336, 1.07), ("fwd", 64, 1, 16384, 512, 0.93), ("fwd", 64, 1, 16384, 768, 1.02), ("fwd", 64, 1, 16384, 1024, 0.98),
    ("dq", 128, 0, 1024, 128, 1.12), ("dq", 128, 0, 1024, 136, 0.78), ("dq", 128, 1, 1024, 192, 1.02), ("dq", 128, 1, 1536, 300, 1.17),
    ("dq", 128, 1, 1024, 384, 0.98), ("dq", 128, 1, 2048, 256, 1.02), ("dq", 128, 1, 2048, 512, 0.96), ("dq", 128, 1, 8192, 160, 1.02),
    ("dq", 128, 1, 2560, 300, 0.99), ("dq", 128, 1, 1280, 450, 0.92), ("dq", 128, 1, 3072, 384, 0.96), ("dq", 64, 0, 1024, 256, 0.91),
    ("dq", 64, 0, 1024, 288, 1.20), ("dq", 64, 1, 2048, 160, 1.09), ("dq", 64, 1, 1024, 288, 1.04), ("dq", 64, 1, 4096, 320, 1.02),
    ("dq", 64, 1, 4096, 384, 0.97), ("dq", 64, 1, 2560, 700, 1.12), ("dq", 64, 1, 8192, 256, 1.04), ("dq", 64, 1, 8192, 384, 0.98),
    ("dkdv64", 64, 0, 1024, 136, 0.85), ("dkdv64", 64, 0, 8192, 320, 1.12), ("dkdv64", 64, 0, 8192, 448, 0.89), ("dkdv64", 64, 0, 1024, 576, 1.08),
    ("dkdv64", 64, 0, 256, 272, 1.06), ("dkdv64", 64, 0, 1280, 540, 1.04), ("dkdv64", 64, 0, 512, 448, 0.95), ("dkdv64", 64, 0, 512, 1024, 0.96),
    ("dkdv64", 64, 0, 768, 465, 0.92), ("dkdv64", 64, 0, 1024, 1024, 0.95),
    ("dkdv64", 64, 1, 2048, 192, 1.12), ("dkdv64", 64, 1, 1024, 288, 1.04), ("dkdv64", 64, 1, 2560, 700, 1.15), ("dkdv64", 64, 1, 4096, 320, 1.04),
    ("dkdv64", 64, 1, 4096, 448, 0.97), ("dkdv64", 64, 1, 8192, 256, 1.09), ("dkdv64", 64, 1, 8192, 512, 0.95)]


@pytest.mark.parametrize("what,d,causal,N,b,ratio", MEASURED)
def test_fixed_length_rules_take_the_faster_kernel(D, what, d, causal, N, b, ratio):
    assert bool(getattr(D, "t_" + what)(d, causal, N, b)) == (ratio < 1)


def test_d256_rules(D):
    assert D.t_dq256(1, 128, 64) and not D.t_dq256(1, 128, 512) and D.t_dq256(0, 128, 512) and D.t_dq256(1, 256, 512)
    assert D.t_dkdv256(128, 64) and not D.t_dkdv256(128, 256) and D.t_dkdv256(512, 256)


# the same for variable lengths: (d, causal, mean queries, mean keys, H, Hkv, tokens, share of the backward pass that dQ and dK/dV
# with one wave per SIMD add)
MEASURED_VARLEN = [
    (128, 1, 16, 16, 16, 8, 16384, 0.52, 0.155), (128, 1, 64, 64, 16, 8, 16384, 0.46, 0.072), (128, 1, 100, 100, 16, 8, 16300, 0.174, -0.096),
    (128, 0, 16, 1000, 16, 8, 512, None, -0.027), (128, 1, 800, 800, 16, 8, 4000, 0.127, -0.03), (128, 1, 1500, 1500, 16, 8, 15000, -0.071, -0.08),
    (128, 0, 512, 512, 16, 8, 4096, -0.127, -0.07), (192, 1, 32, 32, 16, 8, 16384, 0.133, 0.090), (192, 0, 32, 32, 16, 8, 16384, 0.106, -0.225),
    (192, 0, 800, 800, 16, 8, 16000, -0.02, -0.40), (256, 1, 64, 64, 16, 16, 16384, 0.071, 0.320), (256, 1, 64, 4096, 16, 8, 1024, -0.049, 0.197),
    (256, 1, 200, 200, 16, 8, 16200, -0.097, -0.108), (256, 0, 8, 8, 16, 16, 16384, 0.112, 0.056), (256, 0, 64, 64, 16, 8, 16384, 0.077, -0.146),
    (64, 1, 1024, 1024, 16, 8, 16384, 0.110, None), (64, 1, 8192, 8192, 16, 8, 16384, -0.051, -0.092), (64, 1, 8192, 8192, 8, 2, 65536, -0.029, 0.050),
    (64, 0, 2048, 2048, 16, 8, 16384, -0.035, -0.057), (64, 0, 2048, 2048, 4, 4, 16384, 0.043, 0.050)]


@pytest.mark.parametrize("d,causal,n,k,H,Hkv,tokens,dq,dkdv", MEASURED_VARLEN)
def test_varlen_rules_take_the_faster_kernel(D, d, causal, n, k, H, Hkv, tokens, dq, dkdv):
    B = tokens // n
    half, blocks64 = (tokens + 255) // 256 * H, (B * k // 128 + B) // 2 * Hkv
    if dq is not None:
        assert bool(D.t_dq_varlen(d, causal, n, k, half)) == (dq < 0)
    if dkdv is not None:
        assert bool(D.t_dkdv_varlen(d, causal, n, k, H // Hkv, blocks64)) == (dkdv < 0)


# forward, variable lengths: (d, causal, B, queries, keys, H, Hkv, equal lengths, 64-queries-per-wave kernel over 128-row kernel)
MEASURED_FWD_VARLEN = [
    (128, 0, 16, 1500, 1500, 16, 16, 1, 0.95), (192, 0, 16, 1500, 1500, 16, 16, 0, 0.98),
    (192, 0, 24, 1000, 1000, 16, 16, 0, 1.05), (128, 0, 64, 692, 692, 16, 16, 0, 1.10), (128, 1, 8, 3000, 3000, 16, 16, 1, 1.03),
    (128, 1, 4, 4000, 4000, 16, 16, 1, 0.97), (192, 1, 4, 6000, 6000, 16, 16, 1, 0.93), (192, 1, 8, 3000, 3000, 16, 16, 0, 1.03),
    (128, 1, 32, 1160, 1160, 16, 16, 0, 1.07), (128, 1, 1, 4096, 4096, 16, 16, 1, 1.10), (128, 1, 1, 512, 8192, 32, 8, 1, 0.93),
    (128, 1, 1, 512, 32768, 32, 8, 1, 0.86), (192, 1, 2, 512, 8192, 32, 8, 1, 0.87), (128, 1, 1, 512, 8192, 16, 16, 1, 1.02),
    (128, 1, 2, 1024, 3000, 16, 16, 1, 1.05), (128, 0, 2, 1024, 3000, 16, 16, 1, 0.96), (128, 1, 1, 384, 16384, 32, 8, 1, 1.44),
    (192, 1, 1, 640, 16384, 32, 8, 1, 1.40), (192, 1, 2, 300, 6000, 16, 8, 1, 1.52), (192, 1, 4, 300, 8192, 32, 8, 1, 0.90),
    (128, 1, 1, 500, 2000, 64, 64, 1, 1.25), (128, 1, 2, 500, 2000, 64, 64, 1, 0.94), (128, 1, 1, 512, 8192, 32, 8, 0, 0.93)]


@pytest.mark.parametrize("d,causal,B,nq,nk,H,Hkv,equal,ratio", MEASURED_FWD_VARLEN)
def test_varlen_forward_rule_takes_the_faster_kernel(D, d, causal, B, nq, nk, H, Hkv, equal, ratio):
    assert abs(ratio - 1) < 0.01 or bool(D.t_fwd_varlen(d, causal, B, B * nq, B * nk, H, Hkv, equal)) == (ratio < 1)


def test_gpu_tests_that_compare_two_forward_kernels_run_two(D):
    import test_gpu_varlen as V
    for lists, fixed, packed in ((V.SAME_KERNEL, 0, 0), (V.OTHER_KERNEL, 1, 0), (V.BOTH_64, 1, 1)):
        for B, N, causal in lists:
            assert D.t_fwd(128, causal, N, B * 4 * N // 256) == fixed, (B, N, causal)
            assert D.t_fwd_varlen(128, causal, B, B * N, B * N, 4, 2, 0) == packed, (B, N, causal)


def test_gpu_tests_of_the_varlen_forward_kernel_reach_it(D):
    import test_gpu_fwd_varlen_one_wave as W
    parts = set()
    for d, causal, B, nq, nk, H in W.EQUAL:
        assert D.t_fwd_varlen(d, causal, B, B * nq, B * nk, H, H, 1), (d, nq, nk)
        parts.add(route(D, B, B * nq, B * nk, H, H, d, 128, 1)[1])
    for d, causal, lens, H in W.PACKED:
        Tq, Tk = (sum(x[i] for x in lens) for i in (0, 1))
        assert D.t_fwd_varlen(d, causal, len(lens), Tq, Tk, H, H, 0), lens
        parts.add(route(D, len(lens), Tq, Tk, H, H, d, 128, 0)[1])
    assert 1 in parts and len(parts) > 1
    for d, causal, lens, H in W.UNSEEN:
        Tq, Tk = (sum(x[i] for x in lens) for i in (0, 1))
        nsplit = route(D, len(lens), Tq, Tk, H, H, d, 128, 0)[1]
        assert nsplit > 1 and D.t_fwd_varlen(d, causal, len(lens), Tq, Tk, H, H, 0), lens
        # a block whose second part begins past what its first queries see
        assert any(nq >= 256 > nk - nq + 1 and nk > 256 + 64 for nq, nk in lens)
    parts = set()
    for d, causal, B, nq, nk, H, Hkv in W.GROUPED:
        parts.add(route(D, B, B * nq, B * nk, H, Hkv, d, 128, 1)[1])
        assert D.t_fwd_varlen(d, causal, B, B * nq, B * nk, H, Hkv, 1), (d, nq, nk)
    assert 1 in parts and len(parts) > 1
    for d, B, nq, nk, H, key in W.NOT_FINITE:
        fixed = nq == nk and nq % 128 == 0
        assert D.t_fwd(d, 1, nq, B * H * nq // 256) if fixed else D.t_fwd_varlen(d, 1, B, B * nq, B * nk, H, H, 1), (d, nq, nk)


def route(D, B, Tq, Tk, H, Hkv, dqk, dv, uniform):
    """(decode kernel, parts of the keys) of a forward call."""
    nsplit = ctypes.c_int()
    return bool(D.t_route(B, Tq, Tk, H, Hkv, dqk, dv, uniform, ctypes.byref(nsplit))), nsplit.value


@pytest.mark.parametrize("B,Tq,Tk,H,Hkv,d", [(1, 512, 8192, 32, 8, 128), (4, 256, 16384, 32, 8, 128), (8, 1600, 24000, 8, 2, 64),
                                             (2, 400, 13000, 16, 4, 64), (1, 128, 16384, 32, 8, 256)])
def test_merge_of_a_packed_chunk_has_blocks_for_its_rows(D, B, Tq, Tk, H, Hkv, d):
    """Packed sequences of several queries whose keys are divided: every row of a full tile within one turn of a merge block,
    as for the strided call of the same sizes."""
    assert route(D, B, Tq, Tk, H, Hkv, d, d, 0)[1] > 1 and D.t_shares(B, Tq, Tk, H, Hkv, d, d, 0) * (1024 // d) >= 128 * (H // Hkv)


# (B, H, Hkv, Nq, Nk, d, decode kernel over 128-row kernel): both sides of the lines, equal lengths
MEASURED_DECODE = [(256, 16, 16, 1, 64, 64, 1.52), (256, 16, 16, 1, 256, 64, 1.19), (64, 16, 16, 1, 1024, 64, 0.91), (256, 16, 16, 1, 64, 128, 1.13),
                   (256, 16, 16, 1, 320, 128, 0.97), (256, 16, 16, 16, 16, 256, 1.29), (256, 16, 16, 1, 64, 192, 0.95), (4, 16, 8, 1, 64, 64, 1.27),
                   (16, 16, 8, 16, 128, 128, 1.18), (32, 32, 8, 1, 64, 128, 0.59), (512, 16, 4, 16, 16, 192, 0.67), (1, 8, 8, 16, 64, 192, 1.29),
                   (2, 32, 8, 24, 4096, 128, 0.45)]


@pytest.mark.parametrize("B,H,Hkv,Nq,Nk,d,ratio", MEASURED_DECODE)
def test_decode_rule_takes_the_faster_kernel(D, B, H, Hkv, Nq, Nk, d, ratio):
    assert route(D, B, B * Nq, B * Nk, H, Hkv, d, 128 if d == 192 else d, 1)[0] == (ratio < 1)


# (items, Nk, d, three parts over one)
@pytest.mark.parametrize("items,Nk,d,ratio", [(264, 1000, 128, 0.97), (320, 2000, 128, 0.91), (384, 2000, 128, 0.99), (480, 2000, 128, 1.07),
                                              (320, 4000, 128, 0.88), (480, 4000, 128, 1.04), (800, 4000, 128, 0.93), (320, 300, 256, 1.32),
                                              (264, 1000, 256, 0.91), (352, 1000, 256, 1.04), (264, 2000, 64, 0.87), (320, 1000, 64, 1.18),
                                              (448, 4000, 64, 0.97)])
def test_partly_filled_rounds_are_divided_where_it_pays(D, items, Nk, d, ratio):
    """(Within 3 % either choice will do.)"""
    B = items // 8
    decode, nsplit = route(D, B, B, B * Nk, 32, 8, d, d, 1)
    assert decode and (abs(ratio - 1) < 0.035 or nsplit == (3 if ratio < 1 else 1))


# (d, causal, queries, keys, KV heads in all, query heads per KV head, one kernel over two): both sides of the lines
MEASURED_SHORT = [(64, 0, 128, 128, 8, 1, 0.85), (64, 1, 128, 128, 128, 4, 1.22), (64, 1, 128, 128, 512, 4, 0.65), (64, 0, 100, 512, 64, 1, 0.96),
                  (64, 0, 128, 512, 16, 1, 1.02), (64, 0, 160, 256, 16, 1, 1.03), (64, 0, 200, 200, 96, 1, 1.10), (64, 0, 200, 200, 320, 1, 0.72),
                  (64, 0, 256, 256, 96, 1, 1.27), (64, 0, 256, 256, 512, 1, 0.79), (64, 1, 384, 384, 384, 1, 1.14), (64, 1, 512, 512, 256, 1, 0.86),
                  (64, 0, 512, 512, 512, 1, 1.02), (64, 0, 512, 512, 256, 1, 0.90), (64, 0, 4096, 512, 64, 1, 2.47), (64, 0, 4096, 512, 256, 1, 0.85),
                  (96, 0, 160, 256, 16, 1, 0.80), (96, 1, 100, 100, 128, 4, 1.08), (96, 1, 128, 128, 224, 4, 0.81), (96, 0, 256, 256, 128, 4, 1.15),
                  (96, 0, 256, 256, 512, 1, 0.65), (128, 0, 128, 128, 8, 1, 0.87), (128, 0, 100, 100, 128, 4, 1.28), (128, 0, 128, 128, 256, 4, 0.85),
                  (128, 0, 256, 256, 128, 1, 1.11), (128, 0, 256, 256, 256, 1, 0.76), (128, 0, 1000, 77, 256, 1, 1.05), (128, 0, 1000, 77, 1024, 1, 0.72),
                  (128, 1, 256, 256, 512, 8, 0.58)]


@pytest.mark.parametrize("d,causal,nq,nk,blocks,group,ratio", MEASURED_SHORT)
def test_short_backward_rule_takes_the_faster_route(D, d, causal, nq, nk, blocks, group, ratio):
    """(Within 4 % either choice will do.)"""
    assert abs(ratio - 1) < 0.045 or bool(D.t_short(d, causal, nq, nk, 1, blocks * group, blocks)) == (ratio < 1)


# just past a full round of blocks, beside the same call with a round that fills: (d, causal, queries, keys, blocks, heads per KV head, ratio)
@pytest.mark.parametrize("d,causal,nq,nk,blocks,group,ratio", [
    (64, 1, 256, 256, 520, 8, 1.14), (64, 0, 1024, 256, 544, 1, 1.11), (64, 0, 1024, 256, 512, 1, 0.78), (64, 0, 1024, 256, 768, 1, 0.82), (64, 0, 1024, 128, 520, 1, 1.08),
    (64, 0, 100, 100, 520, 2, 0.87), (64, 1, 160, 160, 520, 8, 0.89), (64, 1, 192, 192, 264, 8, 1.08), (64, 0, 4096, 100, 264, 1, 1.11), (64, 0, 4096, 256, 1032, 1, 0.78),
    (96, 1, 256, 256, 264, 8, 1.14), (96, 0, 4096, 256, 320, 1, 1.08), (96, 0, 192, 192, 264, 2, 0.79), (96, 0, 4096, 128, 520, 1, 0.90),
    (128, 0, 4096, 256, 264, 1, 1.16), (128, 1, 192, 192, 264, 8, 0.90), (128, 0, 4096, 224, 264, 1, 1.13), (128, 0, 4096, 256, 256, 1, 0.67), (128, 0, 4096, 256, 520, 1, 0.98),
    (128, 0, 4096, 100, 520, 1, 0.90), (128, 1, 100, 100, 520, 8, 0.80), (128, 0, 4096, 128, 264, 1, 0.82), (64, 0, 300, 300, 776, 1, 1.11), (64, 0, 2048, 300, 776, 1, 0.89), (64, 1, 256, 256, 520, 2, 1.05), (64, 0, 300, 300, 512, 1, 0.85), (64, 1, 450, 450, 1032, 1, 0.93)])
def test_short_backward_rule_leaves_rounds_that_barely_begin(D, d, causal, nq, nk, blocks, group, ratio):
    test_short_backward_rule_takes_the_faster_route(D, d, causal, nq, nk, blocks, group, ratio)


# whole tiles, by the fixed-length call: (d, causal, tokens, blocks, heads per KV head, ratio)
@pytest.mark.parametrize("d,causal,n,blocks,group,ratio", [
    (64, 0, 128, 256, 8, 1.24), (64, 0, 128, 512, 8, 0.94), (64, 0, 128, 544, 4, 1.13), (64, 0, 128, 640, 16, 1.24), (64, 0, 128, 960, 8, 0.95), (64, 0, 128, 320, 4, 0.98),
    (64, 0, 128, 832, 4, 0.97), (64, 1, 128, 640, 4, 0.94), (64, 1, 128, 256, 16, 1.20), (64, 1, 128, 448, 16, 0.90), (64, 1, 128, 544, 8, 1.12), (64, 1, 128, 768, 8, 0.93),
    (64, 0, 256, 544, 2, 1.16), (64, 0, 256, 640, 8, 1.27), (64, 0, 256, 512, 1, 0.79), (64, 0, 256, 1536, 8, 0.92), (64, 1, 256, 320, 8, 1.18), (64, 1, 256, 320, 2, 0.96),
    (64, 1, 256, 768, 4, 0.93), (64, 1, 256, 576, 16, 1.22), (64, 0, 512, 256, 4, 1.06), (64, 0, 512, 256, 1, 0.93), (64, 1, 512, 264, 1, 1.48), (64, 1, 384, 512, 2, 0.97),
    (96, 0, 128, 192, 8, 1.12), (96, 0, 128, 240, 8, 0.96), (96, 1, 256, 264, 2, 1.17), (96, 1, 256, 160, 8, 1.09), (96, 0, 256, 192, 8, 0.85), (128, 0, 128, 256, 16, 1.19),
    (128, 0, 128, 264, 16, 0.96), (128, 0, 128, 528, 16, 1.14), (128, 1, 128, 528, 16, 0.94), (128, 0, 256, 352, 8, 1.20), (128, 1, 256, 352, 2, 0.94), (128, 0, 256, 544, 4, 1.09),
    (128, 1, 256, 192, 8, 0.91), (128, 0, 256, 640, 2, 0.99)])
def test_short_backward_rule_of_whole_tiles(D, d, causal, n, blocks, group, ratio):
    assert bool(D.t_short(d, causal, n, n, 1, blocks * group, blocks)) == (ratio < 1)


def test_short_backward_keys_fit_the_block(D):
    """Never more keys than a block holds, and no other head dims, however many blocks."""
    for d, most in ((64, 512), (96, 256), (128, 256), (192, 0), (256, 0)):
        assert not D.t_short(d, 1, 1, most + 1, 1024, 64, 64) and (most == 0 or D.t_short(d, 1, 1, most, 1024, 64, 64))


# (causal, blocks, rows that a block walks, three blocks per CU over two), d = 64: both sides of the lines
@pytest.mark.parametrize("causal,blocks,loop,ratio", [(0, 512, 1024, 1.02), (0, 528, 384, 0.92), (0, 576, 1000, 0.93), (0, 640, 2000, 0.95), (1, 528, 384, 1.06), (1, 576, 1000, 1.03),
                                                      (1, 640, 2000, 1.05), (1, 704, 1000, 0.93), (1, 1088, 1024, 0.90), (0, 6144, 60, 1.05), (0, 6144, 130, 0.94)])
def test_lean_backward_rule(D, causal, blocks, loop, ratio):
    assert bool(D.t_lean(64, causal, blocks, loop)) == (ratio < 1)
    assert not any(D.t_lean(d, causal, blocks, loop) for d in (96, 128, 192, 256))


# dQ, d = 64: (causal, blocks, queries, keys, three blocks per CU over two)
@pytest.mark.parametrize("causal,blocks,nq,nk,ratio", [(0, 1024, 60, 2000, 1.06), (1, 1024, 60, 2000, 1.05), (1, 1024, 20, 700, 1.02), (0, 1024, 128, 2000, 1.05), (0, 2048, 129, 700, 0.95),
                                                       (1, 2048, 129, 700, 0.90), (0, 768, 300, 2000, 0.93)])
def test_lean_dq_rule(D, causal, blocks, nq, nk, ratio):
    assert bool(D.t_lean_dq(64, causal, blocks, nq, nk)) == (ratio < 1)


# packed, d = 64, no mask: (lengths, heads, three blocks per CU on the room of the tables over two)
@pytest.mark.parametrize("B,T,room,H,lean", [(64, 9856, 141, 4, False), (20, 6016, 67, 8, False), (48, 10752, 132, 4, False), (40, 7800, 101, 8, True), (9, 9000, 79, 8, True),
                                             (24, 7128, 79, 8, True), (30, 4020, 62, 12, True)])
def test_lean_rule_counts_tiles_that_are_there(D, B, T, room, H, lean):
    blocks = D.t_tiles(0, room, T, B) * H
    assert blocks <= room * H and bool(D.t_lean(64, 0, blocks, T // B)) == lean
    assert D.t_tiles(1, room, T, B) == room


@pytest.mark.parametrize("causal,blocks,loop,lean", [(0, 792, 300, False), (0, 800, 600, False), (0, 768, 600, True), (0, 1040, 600, True), (0, 800, 640, True), (1, 800, 600, True)])
def test_lean_rule_past_three_blocks_per_cu(D, causal, blocks, loop, lean):
    assert bool(D.t_lean_strided(causal, blocks, loop)) == lean and D.t_lean(64, causal, blocks, loop)


# (B, H, Hkv, queries, keys, d, parts): one CU per block, parts of four tiles; two per CU, of sixteen; loops too short to divide
@pytest.mark.parametrize("B,H,Hkv,Nq,Nk,d,parts", [(3, 16, 2, 59, 1687, 96, 5), (2, 16, 16, 34, 1359, 256, 5), (1, 32, 8, 512, 8192, 128, 4), (1, 8, 8, 1000, 4000, 128, 4),
                                                   (4, 16, 16, 200, 3000, 128, 2), (4, 32, 8, 100, 4000, 128, 3), (1, 32, 8, 128, 600, 128, 1),
                                                   (1, 16, 16, 500, 700, 128, 1), (16, 16, 4, 100, 1500, 128, 1), (8, 32, 8, 200, 6000, 128, 1)])
def test_parts_of_a_chunk(D, B, H, Hkv, Nq, Nk, d, parts):
    assert route(D, B, B * Nq, B * Nk, H, Hkv, d, d, 1) == (False, parts)


# (B, H, Hkv, keys, d, parts)
@pytest.mark.parametrize("B,H,Hkv,Nk,d,parts", [(4, 8, 8, 1000, 128, 4), (1, 8, 8, 1000, 128, 4), (2, 8, 2, 1316, 96, 5), (2, 8, 8, 2000, 64, 5), (4, 16, 16, 600, 64, 1),
                                                (2, 8, 8, 1000, 256, 8), (16, 32, 8, 1000, 128, 1), (8, 16, 4, 273, 64, 1), (1, 32, 8, 32768, 128, 16)])
def test_parts_of_a_decode_step_of_few_blocks(D, B, H, Hkv, Nk, d, parts):
    assert route(D, B, B, B * Nk, H, Hkv, d, d, 1) == (True, parts)


# (B, H, Hkv, queries, keys, d, parts): few heads against long caches, where the merge counts
@pytest.mark.parametrize("B,H,Hkv,Nq,Nk,d,parts", [(1, 1, 1, 1, 32768, 128, 37), (1, 8, 1, 1, 32768, 64, 32), (1, 1, 1, 1, 32768, 256, 64), (2, 8, 2, 1, 8192, 128, 16), (1, 1, 1, 1, 2300, 256, 18), (1, 8, 8, 1, 3051, 128, 12),
                                                   (1, 4, 4, 1, 8192, 64, 16), (1, 1, 1, 1, 2048, 128, 8), (1, 1, 1, 1, 2048, 256, 16), (6, 16, 16, 1, 826, 128, 1), (10, 2, 2, 1, 792, 64, 1), (2, 16, 16, 1, 826, 128, 3), (2, 32, 32, 1, 500, 256, 1), (1, 32, 8, 1, 32768, 128, 16),
                                                   (1, 1, 1, 64, 32768, 128, 45), (2, 2, 1, 100, 16384, 128, 31), (1, 4, 4, 100, 32768, 96, 45), (1, 1, 1, 64, 32768, 256, 67),
                                                   (1, 4, 4, 300, 8192, 64, 21), (1, 1, 1, 64, 2048, 128, 7)])
def test_parts_of_few_heads_against_long_caches(D, B, H, Hkv, Nq, Nk, d, parts):
    assert route(D, B, B * Nq, B * Nk, H, Hkv, d, d, 1) == (Nq == 1, parts)


def test_parts_of_a_decode_step_hold_keys(D):
    """d = 64: as many parts as the kernel's division into whole steps of four 32-key tiles leaves with keys; other head dims, packed batches and
    chunks as they are."""
    for nk in list(range(1, 1200)) + [2000, 2047, 2049, 8191, 32768, 2 ** 31 - 1]:
        for n in (1, 2, 3, 4, 5, 8, 16, 32, 127):
            tiles = (nk + 31) // 32
            per = ((tiles + n - 1) // n + 3) & ~3
            assert D.t_live(1, 1, 64, nk, n) == -(-tiles // per) and D.t_live(1, 1, 128, nk, n) == n
            assert D.t_live(0, 1, 64, nk, n) == n and D.t_live(1, 0, 64, nk, n) == n


def test_parts_of_a_packed_step(D):
    assert route(D, 3, 1000, 5000, 4, 2, 128, 128, 0) == (False, 1)             # a packed chunk: parts of 16 tiles
    assert route(D, 3, 1000, 10000, 4, 2, 128, 128, 0) == (False, 3)
    assert route(D, 1, 1, 32768, 32, 8, 128, 128, 0) == (True, 16)              # a sequence alone: 128 blocks, not 1024
    assert route(D, 48, 48, 48 * 1700, 32, 8, 128, 128, 0) == (True, 3)
    assert route(D, 512, 512, 512 * 64, 16, 16, 64, 64, 0)[0] is False          # tiny caches of many heads
    assert route(D, 512, 32, 32 * 1000, 16, 16, 64, 64, 0)[0] is True           # (slots without a query do not count)


def test_gpu_tests_reach_what_they_are_written_for(D):
    """The case lists of the GPU tests, through the rules: a kernel's tests stop being its tests when a line moves."""
    import test_gpu_bwd_lean as L
    import test_gpu_bwd_short as K
    import test_gpu_edge as E
    import test_gpu_few_blocks as S
    import test_gpu_fp16 as H
    import test_gpu_fwd as F
    import test_gpu_varlen as V
    import test_gpu_varlen_one_wave as W
    from test_gpu_decode import CHUNKS, FEW_KEYS, SHAPES, SLOTS
    for d, nq, nk, group, Hkv, causal, _ in K.CASES:
        assert D.t_short(d, causal, nq, nk, 1, Hkv * group, Hkv), (d, nq, nk, group, Hkv)
    for d, N, B, causal in K.PASSES:
        assert D.t_short(d, causal, N, N, B, 8, 8), (d, N, B)
    for nq, nk, group, Hkv, causal, _ in L.CASES:
        assert D.t_lean(64, causal, (nk + 127) // 128 * Hkv, nq * group) and not D.t_short(64, causal, nq, nk, 1, Hkv * group, Hkv), (nq, nk, Hkv)
        assert not D.t_lean(64, causal, (nk + 127) // 128 * 2, nq * group) and not D.t_short(64, causal, nq, nk, 1, 2 * group, 2), (nq, nk)
    for w, times in F.Q64 + H.ONE_WAVE:
        assert D.t_fwd(w.dqk, w.causal, w.N, w.B * w.H * times * w.N // 256), w.name
    for causal, N, d, _, times, *_ in F.GROWING + F.STEPS:
        assert D.t_fwd(d, causal, N, 2 * times * N // 256), (causal, N, d)
    for causal, N, heads, d, _ in S.FORWARD + S.FORWARD_4_WAVE:
        assert bool(D.t_fwd(d, causal, N, heads * N // 256)) == ((causal, N, heads, d, d) not in S.FORWARD_4_WAVE), (causal, N, heads, d)
    for causal, N, heads, d in S.BACKWARD + S.BACKWARD_4_WAVE:
        want = (causal, N, heads, d) in S.BACKWARD
        assert bool(D.t_dq(d, causal, N, heads * N // 256)) == want
        assert d != 64 or bool(D.t_dkdv64(d, causal, N, heads * N // 256)) == want
    for causal, d, N, times in E.DQ_TILES:
        assert D.t_dq(d, causal, N, 4 * times * N // 256), (causal, N, d)
    for w, times in H.ONE_WAVE:
        assert w.dqk == 192 or D.t_dq(w.dqk, w.causal, w.N, w.H * times * w.N // 256), w.name
        assert w.dqk != 64 or w.H != w.Hkv or D.t_dkdv64(64, w.causal, w.N, w.Hkv * times * w.N // 256), w.name
    for cases, want in ((V.SAME_KERNEL, False), (V.OTHER_KERNEL, True)):
        for B, N, causal in cases:
            assert bool(D.t_fwd(128, causal, N, B * 4 * N // 256)) == want, (B, N, causal)
    for cases, want in ((V.BWD_SAME, False), (V.BWD_OTHER, True)):
        for dqk, _, _, N, causal, B, heads, Hkv in cases:
            b = B * heads * N // 256
            assert (dqk != 192 and bool(D.t_dq(dqk, causal, N, b))) == want
            assert not D.t_dq_varlen(dqk, causal, N, N, b)                          # (the packed call: the general kernel)
    for d, causal, lens, _ in W.LARGE:
        n, k = (sum(x[i] for x in lens) for i in (0, 1))
        B = len(lens)
        assert D.t_dq_varlen(d, causal, n // B, k // B, (n + 255) // 256 * 16), lens
        assert D.t_dkdv_varlen(d, causal, n // B, k // B, 2, (k // 128 + B) // 2 * 8), lens
        for nq, nk in lens:
            assert not D.t_dq_varlen(d, causal, nq, nk, (nq + 255) // 256 * 2)      # (two heads of one sequence)
    for dqk, _, causal, lens in W.CASES:
        n, k = (sum(x[i] for x in lens) // len(lens) for i in (0, 1))
        assert D.t_dkdv_varlen(dqk, causal, n, k, 2, 1) and (dqk == 128 or D.t_dq_varlen(dqk, causal, n, k, 1)), lens
    for B, H_, Hkv, Nq, Nk, dqk, dv, _ in SHAPES:
        decode, nsplit = route(D, B, B * Nq, B * Nk, H_, Hkv, dqk, dv, 1)
        assert decode == (Nq < 100) and (decode or nsplit > 1), (B, H_, Hkv, Nq, Nk)
    for B, H_, Hkv, Nq, Nk, dqk, dv, _ in FEW_KEYS:
        assert route(D, B, B * Nq, B * Nk, H_, Hkv, dqk, dv, 1) == (False, 1)
    for cases, want in ((CHUNKS, False), (SLOTS, True)):
        for H_, Hkv, dqk, dv, pairs, _ in cases:
            decode, nsplit = route(D, len(pairs), *(sum(p[i] for p in pairs) for i in (0, 1)), H_, Hkv, dqk, dv, 0)
            assert decode == want and (want or nsplit > 1), pairs
