"""GPU tests of the variable-length form of the forward kernel with 64 queries per wave, whole and with the keys divided:
ragged ends, blocks with a few rows, sequences without queries, a diagonal that is not aligned with the tiles, scores that
send it through its second pass, overlapping rows (which it leaves to the 128-row kernel), grouped heads in views, values that are not finite.  Two heads are generated and
repeated, so that the oracle computes two and every repetition has to reproduce their bits."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import LSE_ABS, assert_close

pytestmark = pytest.mark.gpu

# equal lengths: (d_qk, causal, B, queries, keys, H): keys divided by two; whole; without the mask; self-attention; under the mask
EQUAL = [(128, True, 1, 500, 4161, 64), (128, True, 2, 511, 2033, 64), (192, False, 1, 257, 1300, 70), (128, False, 1, 1281, 1281, 26),
         (128, True, 1, 3600, 3600, 18), (192, True, 1, 385, 6001, 40)]
# packed: (d_qk, causal, [(queries, keys)], H): whole; divided, where a short sequence has fewer parts; without the mask
PACKED = [(128, True, [(500, 4000), (1, 3000), (0, 50), (700, 2900), (257, 3777)], 64), (128, True, [(300, 5000), (513, 6500), (30, 130)], 24),
          (192, False, [(1300, 1300), (129, 1200), (64, 2000), (1000, 700)], 32)]


# packed, divided, under the mask: blocks whose second part of the keys begins past what their first queries see (none, then all of a wave)
UNSEEN = [(128, True, [(300, 7000), (256, 406), (513, 9000)], 20), (192, True, [(700, 8001), (257, 400)], 24)]
# grouped heads: (d_qk, causal, B, queries, keys, H, Hkv): divided, whole, without the mask
GROUPED = [(128, True, 1, 500, 8100, 32, 8), (192, True, 1, 385, 6001, 40, 10), (128, True, 1, 3600, 3600, 18, 6), (128, False, 2, 1281, 1281, 16, 2)]


def _inputs(d, nq, nk, kind, dtype, seed):
    g = torch.Generator("cpu").manual_seed(seed)
    q, k, v = (torch.randn(n, 2, e, generator=g) for n, e in ((nq, d), (nk, d), (nk, 128)))
    if kind == "growing":        # by hundreds of binary orders: relative to the first tile the exponentials overflow
        q, k = q.abs(), k.abs() * torch.linspace(0.2, 30.0, nk).view(nk, 1, 1)
    if kind == "climbing":       # by 300 binary orders in small steps
        q, k = 1.0 + 0.1 * q, torch.linspace(0.0, 300.0 / (1.4427 * d ** 0.5), nk).view(nk, 1, 1) + 0.1 * k
    return [t.to(dtype) for t in (q, k, v)]


def _check(oracle, q, k, v, o, lse, d, causal, what):
    """One sequence: q [n, 2, d], k, v [m, 2, .], o [n, H, 128], lse [H, n]."""
    n, H = o.shape[:2]
    assert all(torch.equal(o[:, h], o[:, h % 2]) and torch.equal(lse[h], lse[h % 2]) for h in range(H)), what
    rows = np.unique(np.concatenate([np.arange(0, n, 37), np.arange(max(0, n - 70), n), np.arange(min(n, 70))]))
    pos = rows + (k.shape[0] - n)
    ro, rlse = oracle.attn_fwd(*(I.to_f64(t[None]) for t in (q[rows], k, v)), d ** -0.5, causal, q_pos=pos)
    assert_close(o[rows, :2][None].float().cpu().numpy(), ro, f"O {what}")
    # (half an ulp of an fp32 LSE above 1024 is 6e-5, above 8192 5e-4)
    assert np.abs(lse[:2].cpu().numpy()[:, rows] - rlse[0]).max() <= LSE_ABS * max(1.0, np.abs(rlse).max() / 64), what


@pytest.mark.parametrize("d,causal,B,nq,nk,H", EQUAL)
@pytest.mark.parametrize("kind,dtype", [("normal", torch.bfloat16), ("growing", torch.bfloat16), ("climbing", torch.bfloat16),
                                        ("normal", torch.float16), ("climbing", torch.float16)])
def test_equal_lengths(oracle, d, causal, B, nq, nk, H, kind, dtype):
    import paper_2603_05451_amd as A
    q, k, v = _inputs(d, nq, nk, kind, dtype, 500 + d + nq)
    rep = lambda t: t.repeat(1, H // 2, 1)[None].repeat(B, 1, 1, 1).cuda()
    room = lambda t: torch.cat([t, torch.full_like(t[:, :64], float("nan"))], 1)[:, :nk]       # keys behind the last are not read
    o, lse = A.attn_fwd_strided(rep(q), room(rep(k)), room(rep(v)), d ** -0.5, causal)
    torch.cuda.synchronize()
    for b in range(B):
        _check(oracle, q, k, v, o[b], lse[b], d, causal, f"{kind} {b}")


@pytest.mark.parametrize("d,causal,lens,H", PACKED)
@pytest.mark.parametrize("kind,dtype", [("normal", torch.bfloat16), ("growing", torch.bfloat16), ("normal", torch.float16)])
def test_packed(oracle, d, causal, lens, H, kind, dtype):
    import paper_2603_05451_amd as A
    x = [_inputs(d, nq, nk, kind, dtype, 540 + d + i) for i, (nq, nk) in enumerate(lens)]
    cu = [torch.tensor(np.concatenate([[0], np.cumsum([n[i] for n in lens])]), dtype=torch.int32, device="cuda") for i in (0, 1)]
    q, k, v = (torch.cat([s[i] for s in x]).repeat(1, H // 2, 1).cuda() for i in range(3))
    o = torch.full(q.shape[:2] + (128,), float("nan"), dtype=dtype, device="cuda")
    _, lse = A.attn_varlen_fwd(q, k, v, cu[0], d ** -0.5, causal, o=o, cu_seqlens_k=cu[1])
    torch.cuda.synchronize()
    at = 0
    for i, (nq, nk) in enumerate(lens):
        if nq:
            _check(oracle, *x[i], o[at:at + nq], lse[:, at:at + nq], d, causal, f"{kind} sequence {i}")
        at += nq


@pytest.mark.parametrize("d,causal,lens,H", UNSEEN)
@pytest.mark.parametrize("kind,dtype", [("normal", torch.bfloat16), ("growing", torch.bfloat16), ("normal", torch.float16)])
def test_parts_that_some_queries_see_nothing_of(oracle, d, causal, lens, H, kind, dtype):
    test_packed(oracle, d, causal, lens, H, kind, dtype)


@pytest.mark.parametrize("d,causal,B,nq,nk,H,Hkv", GROUPED)
@pytest.mark.parametrize("layout", ["bhnd", "fused"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_grouped_heads_in_views(oracle, d, causal, B, nq, nk, H, Hkv, layout, dtype):
    """[B, heads, N, d] storage of Q, K, V and O, and Q beside K and V beside each other in wider buffers with O inside one: the
    bits of contiguous tensors, and the oracle's values.  Every KV head holds one of two, every query head of a group likewise."""
    import paper_2603_05451_amd as A
    q, k, v = _inputs(d, nq, nk, "normal", dtype, 560 + d + nq)
    q = q.repeat(1, H // 2, 1)[None].repeat(B, 1, 1, 1).cuda()
    k, v = (t.repeat(1, Hkv // 2, 1)[None].repeat(B, 1, 1, 1).cuda() for t in (k, v))
    ro, rlse = A.attn_fwd_strided(q, k, v, d ** -0.5, causal)
    if layout == "bhnd":
        view = lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)
        wq, wk, wv = view(q), view(k), view(v)
        o = torch.full((B, H, nq, 128), 7.0, dtype=dtype, device="cuda").transpose(1, 2)
    else:
        wide = lambda t, e: torch.full(t.shape[:2] + (t.shape[2] + 1, e), 7.0, dtype=dtype, device="cuda")
        bq, bkv, bo = wide(q, d), torch.full((B, nk, 2 * Hkv, 192), 7.0, dtype=dtype, device="cuda"), wide(q, 128)
        wq, wk, wv, o = bq[:, :, 1:], bkv[:, :, :Hkv, :d], bkv[:, :, Hkv:, :128], bo[:, :, :H]
        wq.copy_(q); wk.copy_(k); wv.copy_(v)
    _, lse = A.attn_fwd_strided(wq, wk, wv, d ** -0.5, causal, o=o)
    torch.cuda.synchronize()
    assert torch.equal(o, ro) and torch.equal(lse, rlse)
    if layout == "fused":
        assert (bo[:, :, H:] == 7.0).all()
    # query head h meets KV head h / (H / Hkv): the pairs (0, 0) and (G, 1) with G = H / Hkv, and where G is odd (1, 0) ...
    G = H // Hkv
    for h in (0, G, H - 1):
        one = lambda t, i: t[:1, :, i:i + 1].float().cpu().to(dtype)
        rows = np.unique(np.concatenate([np.arange(0, nq, 53), np.arange(max(0, nq - 40), nq)]))
        x = (one(q, h)[:, rows], one(k, h // G), one(v, h // G))
        xo, xl = oracle.attn_fwd(*(I.to_f64(t) for t in x), d ** -0.5, causal, q_pos=rows + (nk - nq))
        assert_close(o[:1, rows, h:h + 1].float().cpu().numpy(), xo, f"O head {h}")
        assert np.abs(lse[:1, h:h + 1].cpu().numpy()[:, :, rows] - xl).max() <= LSE_ABS


def test_overlapping_rows(oracle):
    """Keys and values that are windows of one buffer, 64 elements apart: rows longer than their stride."""
    import paper_2603_05451_amd as A
    nq, nk, H = 511, 2033, 128
    g = torch.Generator("cpu").manual_seed(590)
    q = torch.randn(nq, 2, 128, generator=g).bfloat16()
    base = torch.randn(2, nk * 64 + 64, generator=g).bfloat16()
    k, v = (torch.as_strided(base, (nk, 2, 128), (64, base.shape[1], 1)) for _ in range(2))
    gb = base.repeat(H // 2, 1).cuda()
    gk = torch.as_strided(gb, (1, nk, H, 128), (gb.numel(), 64, gb.shape[1], 1))
    o, lse = A.attn_fwd_strided(q.repeat(1, H // 2, 1)[None].cuda(), gk, gk, 128 ** -0.5, True)
    torch.cuda.synchronize()
    _check(oracle, q, k.contiguous(), v.contiguous(), o[0], lse[0], 128, True, "overlapping")


# (d_qk, B, queries, keys, H, key): divided; self-attention whole; the fixed-length form; a later part that begins past the first queries' diagonal
NOT_FINITE = [(128, 1, 500, 4161, 64, 4160), (128, 1, 500, 4161, 64, 3900), (192, 1, 385, 6001, 40, 5990), (128, 1, 3600, 3600, 18, 3400),
              (128, 1, 6144, 6144, 12, 6000), (192, 2, 6144, 6144, 6, 255)]


@pytest.mark.parametrize("d,B,nq,nk,H,key", NOT_FINITE)
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_values_that_are_not_finite_stay_near_their_diagonal(oracle, d, B, nq, nk, H, key, value, dtype):
    """A row of V that is infinite or NaN reaches the queries that see it and, as 0 * inf, at most those whose 32-query block has its
    64-key tile in its loop: fewer than 95 before them, not the 256 of a block."""
    import paper_2603_05451_amd as A
    q, k, v = _inputs(d, nq, nk, "normal", dtype, 600 + d + nq)
    bad = v.clone()
    bad[key, :, 5] = value
    rep = lambda t: t.repeat(1, H // 2, 1)[None].repeat(B, 1, 1, 1).cuda()
    o, lse = A.attn_fwd_strided(rep(q), rep(k), rep(bad), d ** -0.5, True)
    torch.cuda.synchronize()
    shift = nk - nq
    first = max(0, key - shift)                                     # first query that sees the key
    near = min((q0 for q0 in range(0, nq, 32) if key // 64 * 64 <= q0 + 31 + shift), default=nq)
    assert first - near < 95
    assert torch.isfinite(o[:, :near]).all() and torch.isfinite(lse).all()
    assert not torch.isfinite(o[:, first:, :, 5]).any()
    assert torch.isfinite(torch.cat([o[..., :5], o[..., 6:]], 3)).all()
    ro, rlse = oracle.attn_fwd(*(I.to_f64(t[None]) for t in (q[max(0, near - 300):near], k, v)), d ** -0.5, True,
                               q_pos=np.arange(max(0, near - 300), near) + shift) if near else (None, None)
    if near:
        assert_close(o[:1, max(0, near - 300):near, :2].float().cpu().numpy(), ro, "O before the row")
        assert np.abs(lse[:1, :2, max(0, near - 300):near].cpu().numpy() - rlse).max() <= LSE_ABS
