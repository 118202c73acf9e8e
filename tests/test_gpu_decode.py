"""GPU tests of the forward pass with few queries per sequence against many keys: the decode kernel (the
query heads of a KV head as rows of one tile, keys divided over waves and over blocks), and the 128-row
kernel with its key loop divided over blocks (a chunk of queries against a long cache).  Everything against
the fp64 oracle; sizes sit at the edges of the 32-key tiles, of the rounds of four waves and of the splits."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import LSE_ABS, assert_close

pytestmark = pytest.mark.gpu


def _case(B, H, Hkv, Nq, Nk, dqk, dv, causal, seed, f16=False):
    x = I.make_inputs(I.Workload("decode", B, H, Hkv, max(Nq, Nk), dqk, dv, causal, seed), with_do=False)
    x = {n: t[:, :(Nq if n == "q" else Nk)].contiguous() for n, t in x.items()}
    return {n: t.float().to(torch.float16) for n, t in x.items()} if f16 else x


def _check(oracle, x, o, lse, scale, causal, name):
    Nq, Nk = x["q"].shape[1], x["k"].shape[1]
    ro, rlse = oracle.attn_fwd(*(I.to_f64(x[n]) for n in ("q", "k", "v")), scale, causal, q_pos=np.arange(Nq) + (Nk - Nq))
    assert np.abs(lse.cpu().numpy() - rlse).max() <= LSE_ABS, name
    assert_close(o.float().cpu().numpy(), ro, name)


# (B, H, Hkv, Nq, Nk, d_qk, d_v, causal): one key; around one tile and one round of the four waves; every head
# dim; two queries whose last keys lie in different tiles; two 32-row groups; 64 heads on one KV head; few
# sequences with long caches (many splits, the last of them empty or ragged); chunks with a divided key loop
SHAPES = [(40, 8, 2, 1, 1, 64, 64, True), (40, 8, 1, 1, 31, 128, 128, True), (33, 8, 2, 1, 33, 96, 96, False),
          (2, 4, 4, 1, 127, 192, 128, True), (1, 8, 2, 1, 129, 256, 256, True), (33, 8, 4, 2, 65, 128, 128, True),
          (2, 8, 1, 3, 130, 64, 64, True), (1, 64, 1, 1, 515, 128, 128, True), (2, 16, 4, 10, 300, 128, 128, True),
          (1, 2, 2, 1, 8200, 128, 128, True), (1, 4, 2, 1, 5121, 64, 64, False), (1, 2, 1, 5, 4100, 192, 128, True),
          (1, 2, 1, 2, 3077, 256, 256, True), (1, 3, 3, 1, 2600, 96, 96, True),
          (1, 2, 2, 200, 4161, 128, 128, True), (1, 2, 1, 130, 3300, 64, 64, False), (1, 2, 1, 129, 2500, 256, 256, True),
          (1, 2, 1, 300, 2900, 192, 128, True), (2, 1, 1, 140, 2300, 96, 96, True)]

# as few queries against so few keys that the 128-row kernel keeps them
FEW_KEYS = [(1, 2, 2, 1, 1, 64, 64, True), (3, 4, 1, 1, 31, 128, 128, True), (2, 8, 2, 1, 33, 96, 96, False), (2, 4, 2, 2, 65, 128, 128, True),
            (20, 16, 16, 20, 130, 64, 64, True)]


@pytest.mark.parametrize("shape", SHAPES + FEW_KEYS, ids=["B%d_H%d_%d_q%d_k%d_d%d_%d_%s" % s for s in SHAPES + FEW_KEYS])
def test_few_queries_against_many_keys(oracle, shape):
    import paper_2603_05451_amd as A
    B, H, Hkv, Nq, Nk, dqk, dv, causal = shape
    x = _case(*shape, seed=700 + Nk, f16=Nk % 2 == 0)
    cache = lambda t: torch.cat([t, torch.full_like(t[:, :32], float("nan"))], 1).cuda()[:, :t.shape[1]]    # room behind it
    q, k, v = x["q"].cuda(), cache(x["k"]), cache(x["v"])
    o, lse = A.attn_fwd_strided(q, k, v, dqk ** -0.5, causal)
    # the least workspace a call accepts: fewer parts of the keys, the same result
    nt = lambda n: -(-(B * n // 128 + B) * 32 // 256) * 256
    ws = torch.empty(2 * 256 + nt(Nq), dtype=torch.uint8, device="cuda")
    o1, lse1 = A.attn_fwd_strided(q, k, v, dqk ** -0.5, causal, workspace=ws)
    torch.cuda.synchronize()
    _check(oracle, x, o, lse, dqk ** -0.5, causal, "divided")
    _check(oracle, x, o1, lse1, dqk ** -0.5, causal, "whole")


# a few heads against long caches, in as many parts as the merge pays for: decode steps with and without empty parts, chunks
MANY_PARTS = [(1, 1, 1, 1, 32768, 128, 128, True), (1, 2, 1, 1, 20011, 64, 64, True), (1, 1, 1, 2, 9000, 256, 256, True), (1, 1, 1, 64, 32768, 128, 128, True),
              (1, 2, 1, 100, 9001, 64, 64, False)]


@pytest.mark.parametrize("shape", MANY_PARTS, ids=["B%d_H%d_%d_q%d_k%d_d%d_%d_%s" % s for s in MANY_PARTS])
def test_many_parts(oracle, shape):
    test_few_queries_against_many_keys(oracle, shape)


@pytest.mark.parametrize("H,Hkv,d,lens", [(8, 2, 128, (700, 1, 64, 0, 33, 5000)), (4, 4, 64, (31, 32, 2000)),
                                          (64, 1, 256, (129, 400)), (6, 3, 96, (1500, 96, 5))])
def test_packed_decode_step(oracle, H, Hkv, d, lens):
    """One query per sequence against packed caches of mixed lengths; the sequence without keys has no query."""
    import paper_2603_05451_amd as A
    cuk = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cuq = np.concatenate([[0], np.cumsum([n > 0 for n in lens])]).astype(np.int32)
    x = _case(1, H, Hkv, int(cuq[-1]), int(cuk[-1]), d, d, False, seed=720 + d)
    q, k, v = (x[n][0].cuda() for n in ("q", "k", "v"))
    o, lse = A.attn_varlen_fwd(q, k, v, torch.from_numpy(cuq).cuda(), d ** -0.5, True, cu_seqlens_k=torch.from_numpy(cuk).cuda())
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        if n:
            s = slice(int(cuq[b]), int(cuq[b + 1]))
            part = {"q": x["q"][:, s], "k": x["k"][:, cuk[b]:cuk[b + 1]], "v": x["v"][:, cuk[b]:cuk[b + 1]]}
            _check(oracle, part, o[None, s], lse[None, :, s], d ** -0.5, True, f"sequence {b}")


def _packed_check(oracle, H, Hkv, dqk, dv, pairs, causal, seed, f16=False, **buffers):
    """attn_varlen_fwd of sequences of (queries, keys), every row against the oracle."""
    import paper_2603_05451_amd as A
    cuq, cuk = (np.concatenate([[0], np.cumsum([p[i] for p in pairs])]).astype(np.int32) for i in (0, 1))
    x = _case(1, H, Hkv, int(cuq[-1]), int(cuk[-1]), dqk, dv, False, seed, f16)
    q, k, v = (x[n][0].cuda() for n in ("q", "k", "v"))
    o = torch.full((int(cuq[-1]), H, dv), float("nan"), dtype=q.dtype, device="cuda")
    o, lse = A.attn_varlen_fwd(q, k, v, torch.from_numpy(cuq).cuda(), dqk ** -0.5, causal, o=o,
                               cu_seqlens_k=torch.from_numpy(cuk).cuda(), **buffers)
    torch.cuda.synchronize()
    for b, (nq, nk) in enumerate(pairs):
        if nq:
            sq, sk = slice(int(cuq[b]), int(cuq[b + 1])), slice(int(cuk[b]), int(cuk[b + 1]))
            part = {"q": x["q"][:, sq], "k": x["k"][:, sk], "v": x["v"][:, sk]}
            _check(oracle, part, o[None, sq], lse[None, :, sq], dqk ** -0.5, causal, f"sequence {b}")


# chunks of several queries against a few thousand keys each: the 128-row kernel with its key loop divided.  Whole and ragged tiles,
# a chunk of one query, a sequence without queries, one whose first parts hold all its keys
CHUNKS = [(8, 2, 128, 128, [(200, 5000), (64, 3333), (1, 2500)], True), (4, 4, 64, 64, [(129, 4161), (0, 30), (300, 4500)], False),
          (2, 1, 256, 256, [(130, 2700), (5, 2600)], True), (4, 1, 192, 128, [(128, 4100), (300, 2900), (17, 40)], True)]


@pytest.mark.parametrize("H,Hkv,dqk,dv,pairs,causal", CHUNKS, ids=["d%d_%d" % (c[2], len(c[4])) for c in CHUNKS])
def test_packed_chunks_with_divided_keys(oracle, H, Hkv, dqk, dv, pairs, causal):
    _packed_check(oracle, H, Hkv, dqk, dv, pairs, causal, 750 + dqk, f16=dqk == 64)


def _slots(n, chunks):
    """n slots, most of them empty (with and without keys); chunks: {slot: (queries, keys)}."""
    return [chunks.get(i, (0, 40 if i % 3 == 0 else 0)) for i in range(n)]


# no more queries than sequences, yet sequences of many: a chunk of more than a tile among empty slots, two queries, one; 64 heads on
# one KV head (two 32-row groups per query); three heads (10 rows per turn of the merge kernel at d = 96); keys divided (few slots' worth
# of items) and whole
SLOTS = [(8, 2, 128, 128, _slots(160, {7: (130, 700), 8: (2, 33), 20: (1, 5), 159: (1, 900)}), True),
         (4, 2, 64, 64, _slots(300, {0: (257, 300), 299: (3, 1)}), False), (64, 1, 256, 256, _slots(40, {3: (33, 515), 30: (2, 64)}), True),
         (6, 2, 96, 96, _slots(20, {1: (11, 3000), 2: (5, 700)}), True), (8, 1, 192, 128, _slots(24, {23: (24, 2100)}), True)]


@pytest.mark.parametrize("H,Hkv,dqk,dv,pairs,causal", SLOTS, ids=["d%d_%d" % (c[2], len(c[4])) for c in SLOTS])
def test_chunks_among_empty_slots(oracle, H, Hkv, dqk, dv, pairs, causal):
    _packed_check(oracle, H, Hkv, dqk, dv, pairs, causal, 780 + dqk, f16=dqk in (64, 192))


def test_every_query_of_a_slot_is_listed_once():
    """The table of query tiles with no more queries than sequences: behind the tiles one entry for every query of a tile but its
    first, zeros behind those.  Boundaries that overlap list more queries than there is room for: such a sequence is not listed, its
    tiles' own blocks take all rows, and the results are those of sound boundaries."""
    import paper_2603_05451_amd as A
    from test_gpu_varlen import read_tables
    USED, HELP = 0x5A17AB1E, 0x5A17AB1F
    lens = [0] * 200 + [130, 0, 1, 2, 0, 7] + [0] * 40 + [1] * 3 + [0] * 20          # the longest in another wave than the short ones
    B, cuq = len(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cuk = np.arange(B + 1, dtype=np.int32) * 50
    Tq, Tk = int(cuq[-1]), int(cuk[-1])
    ws = torch.full((A.attn_varlen_workspace_bytes(B, Tq, Tk, 1, 1, 64, 64, True),), 0xAB, dtype=torch.uint8, device="cuda")
    A.attn_varlen_plan(torch.from_numpy(cuq).cuda(), Tq, Tk, 1, 1, 64, 64, ws, cu_seqlens_k=torch.from_numpy(cuk).cuda())
    torch.cuda.synchronize()
    table, _ = read_tables(ws, B, Tq, Tk)
    used = int((table[:, 5] == USED).sum())
    assert (table[:used, 5] == USED).all() and used == sum((n + 127) // 128 for n in lens)
    listed = []
    for e in table[used:Tq]:
        assert e[5] == HELP and 0 <= e[0] < used and table[e[0], 7] == 1 and (e[2:5] == 0).all() and (e[6:] == 0).all()
        listed.append((int(table[e[0], 0]), 128 * int(table[e[0], 4]) + int(e[1])))
    want = [(int(cuq[b]), i) for b, n in enumerate(lens) for i in range(n) if i % 128]
    assert sorted(listed) == sorted(want) and (table[Tq:] == 0).all()
    assert all(t[7] == (min(t[1] - 128 * t[4], 128) > 1 or t[1] > 128) for t in table[:used])

    H, Hkv, d, n = 8, 1, 128, 16
    x = _case(1, H, Hkv, n, 700, d, d, False, 790)
    q, k, v = (x[m][0].cuda() for m in ("q", "k", "v"))
    cu = lambda *c: torch.tensor(c, dtype=torch.int32, device="cuda")
    sound = A.attn_varlen_fwd(q, k, v, cu(0, n, *[n] * (n - 1)), 0.1, True, cu_seqlens_k=cu(0, 700, *[700] * (n - 1)))
    twice = [torch.full_like(t, float("nan")) for t in sound]
    A.attn_varlen_fwd(q, k, v, cu(0, n, 0, n, *[n] * (n - 3)), 0.1, True, o=twice[0], lse=twice[1],
                      cu_seqlens_k=cu(0, 700, 0, 700, *[700] * (n - 3)))
    torch.cuda.synchronize()
    assert torch.equal(sound[0], twice[0]) and torch.equal(sound[1], twice[1])


def test_decode_replays_in_a_graph_and_skips_what_is_not_planned():
    """A captured decode step on new queries gives the eager call's bits; on a workspace without tables a call
    that relies on them leaves its outputs alone, the merge kernel included."""
    import paper_2603_05451_amd as A
    B, H, Hkv, Nk, d = 2, 8, 2, 3000, 128
    x = _case(B, H, Hkv, 1, Nk, d, d, True, seed=740)
    q, k, v = (x[n].cuda() for n in ("q", "k", "v"))
    ws = torch.zeros(A.attn_strided_workspace_bytes(B, H, Hkv, 1, Nk, d, d, False), dtype=torch.uint8, device="cuda")
    o, lse = torch.empty_like(q), torch.empty(B, H, 1, device="cuda")
    A.attn_fwd_strided(q, k, v, 0.1, True, o=o, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        A.attn_fwd_strided(q, k, v, 0.1, True, o=o, lse=lse, workspace=ws, stream=torch.cuda.current_stream())
    for i in range(3):
        q.copy_(torch.randn(q.shape, generator=torch.Generator().manual_seed(i)).bfloat16())
        graph.replay()
        torch.cuda.synchronize()
        ro, rl = A.attn_fwd_strided(q, k, v, 0.1, True)
        assert torch.equal(o, ro) and torch.equal(lse, rl)
    n = A.attn_varlen_workspace_bytes(B, B, B * Nk, H, Hkv, d, d, False)
    o.fill_(7.0)
    lse2 = torch.full((H, B), 7.0, device="cuda")
    A.attn_varlen_fwd(q[:, 0], k.flatten(0, 1), v.flatten(0, 1), None, 0.1, True, o=o[:, 0], lse=lse2, B=B,
                      workspace=torch.zeros(n, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert (o == 7.0).all() and (lse2 == 7.0).all()


# (queries, keys) of at most 64 slots, no more queries than slots: a batch of one, a full wave with equal and unequal keys, empty slots and
# slots without keys, chunks among them, one chunk of all queries, every slot empty but one
FEW = [[(1, 700)], [(1, 100 + 37 * (i % 9)) for i in range(64)], [(1, 1 + 61 * i) for i in range(33)],
       [(0, 40), (3, 500), (1, 0), (0, 0), (2, 129), (1, 4000), (0, 7), (1, 1), (0, 0)], [(0, 5)] * 31 + [(33, 900)] + [(0, 0)] * 3, [(0, 0)] * 20 + [(1, 77)]]


@pytest.mark.parametrize("lens", FEW, ids=[str(len(x)) + "_" + str(sum(n[0] for n in x)) for x in FEW])
@pytest.mark.parametrize("H,Hkv,d", [(8, 2, 128), (4, 4, 64)])
def test_table_of_a_few_sequences(lens, H, Hkv, d):
    """A step of at most 64 sequences finds its table entries in the decode kernel: the bits of a call on the table kernel's
    tables, the same entries left in the workspace (in another order among sequences of one loop length), and those good for a
    call without boundaries."""
    import paper_2603_05451_amd as A
    from test_gpu_varlen import read_tables
    B = len(lens)
    cu = [torch.tensor(np.concatenate([[0], np.cumsum([n[i] for n in lens])]), dtype=torch.int32, device="cuda") for i in (0, 1)]
    Tq, Tk = int(cu[0][-1]), int(cu[1][-1])
    g = torch.Generator(device="cuda").manual_seed(800 + B)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").bfloat16() for n, h in ((Tq, H), (Tk, Hkv), (Tk, Hkv)))
    size = A.attn_varlen_workspace_bytes(B, Tq, Tk, H, Hkv, d, d, True)
    planned, ws = torch.zeros(size, dtype=torch.uint8, device="cuda"), torch.full((size,), 0xCD, dtype=torch.uint8, device="cuda")
    A.attn_varlen_plan(cu[0], Tq, Tk, H, Hkv, d, d, planned, cu_seqlens_k=cu[1])
    out = []
    for c, w in ((None, planned), (cu[0], ws), (None, ws)):
        o, lse = torch.full_like(q, 7.0), torch.full((H, Tq), 7.0, device="cuda")
        A.attn_varlen_fwd(q, k, v, c, 0.1, False, o=o, lse=lse, workspace=w, cu_seqlens_k=None if c is None else cu[1], B=B)
        torch.cuda.synchronize()
        out.append((o, lse))
    assert all(torch.equal(a, b) for other in out[1:] for a, b in zip(out[0], other))
    want, got = (read_tables(w, B, Tq, Tk)[0] for w in (planned, ws))

    def entries(t):         # helpers by their query, whatever the place of its tile
        return sorted(tuple(t[e[0], :4]) + (int(e[1]), 1) if e[5] == 0x5A17AB1F else tuple(e[:4]) + tuple(e[4:]) for e in t)
    assert entries(got) == entries(want)
    keys = [e[3] for e in got if e[5] == 0x5A17AB1E]
    assert keys == sorted(keys, reverse=True)


@pytest.mark.parametrize("B,Nk,parts", [(64, 700, 1), (40, 2600, 3)])
@pytest.mark.parametrize("side", ["k", "q", "both", "decreasing"])
def test_few_sequences_outside_the_tensors_are_left_out(B, Nk, parts, side):
    """Boundaries that run past the stated totals, or decrease, in a step whose table the decode kernel makes itself: that sequence
    is not read or written, the others come out bit for bit as in the sound call."""
    import paper_2603_05451_amd as A
    from test_gpu_varlen import read_tables
    H, Hkv, d = 8, 2, 128
    g = torch.Generator(device="cuda").manual_seed(830 + B)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").bfloat16() for n, h in ((B, H), (B * Nk, Hkv), (B * Nk, Hkv)))
    good = [torch.arange(B + 1, dtype=torch.int32, device="cuda") * n for n in (1, Nk)]
    ws = torch.zeros(A.attn_varlen_workspace_bytes(B, B, B * Nk, H, Hkv, d, d, True), dtype=torch.uint8, device="cuda")
    o_ref, lse_ref = A.attn_varlen_fwd(q, k, v, good[0], 0.1, True, cu_seqlens_k=good[1])
    cq, ck = good[0].clone(), good[1].clone()
    if side in ("k", "both"):
        ck[B] += 64
    if side in ("q", "both"):
        cq[B] += 3
    if side == "decreasing":
        ck[B] = 0
    o, lse = torch.full_like(o_ref, 7.0), torch.full_like(lse_ref, 7.0)
    A.attn_varlen_fwd(q, k, v, cq, 0.1, True, o=o, lse=lse, workspace=ws, cu_seqlens_k=ck)
    torch.cuda.synchronize()
    assert torch.equal(o[:-1], o_ref[:-1]) and torch.equal(lse[:, :-1], lse_ref[:, :-1])
    assert (o[-1] == 7.0).all() and (lse[:, -1] == 7.0).all()
    table = read_tables(ws, B, B, B * Nk)[0]
    assert sorted(t[6] for t in table if t[5] == 0x5A17AB1E) == list(range(B - 1))
