"""GPU tests of the variable-length forms of the backward kernels with one wave per SIMD (64 or 32 queries per
wave for dQ, 32-query tiles for dK/dV): ragged ends inside a 32-row tile, odd numbers of 128-row tiles, a
diagonal that is not aligned with the tiles, overlapping rows.  Mean lengths put the calls on these kernels;
everything against the fp64 oracle, every row and key."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import assert_close, dq_bound_of_one_ds_ulp, half_ulp

pytestmark = pytest.mark.gpu

# (d_qk, d_v, causal, [(queries, keys)]): ends 1, 31, 32, 33 rows into a tile, just below and above 128 and 256,
# one sequence that is a single row; keys - queries a multiple of 128, of 32, of neither
CASES = [(128, 128, True, [(513, 513), (1055, 1055), (300, 300), (896, 896)]),
         (128, 128, False, [(257, 1000), (1025, 95), (640, 640)]),
         (128, 128, True, [(1, 700), (545, 673), (1100, 1133), (700, 1499), (383, 384)]),
         (192, 128, True, [(1153, 1153), (1023, 1200), (1000, 1065)]),
         (192, 128, False, [(545, 300), (500, 1057)]),
         (256, 256, True, [(513, 513), (1, 300), (300, 333), (257, 384)]),
         (256, 256, False, [(129, 700), (385, 95)])]


@pytest.mark.parametrize("dqk,dv,causal,lens", CASES, ids=["d%d_%s_%d" % (c[0], "c" if c[2] else "nc", len(c[3])) for c in CASES])
@pytest.mark.parametrize("f16", [False, True])
def test_packed_backward_of_every_row(oracle, dqk, dv, causal, lens, f16):
    import paper_2603_05451_amd as A
    H, Hkv = 2, 1
    cuq, cuk = (np.concatenate([[0], np.cumsum([x[i] for x in lens])]).astype(np.int32) for i in (0, 1))
    x = I.make_inputs(I.Workload("ow", 1, H, Hkv, int(max(cuq[-1], cuk[-1])), dqk, dv, causal, 760 + dqk + len(lens)))
    if f16:
        x = {n: t.float().to(torch.float16) for n, t in x.items()}
    t = {n: x[n][0, :int((cuq if n in ("q", "do") else cuk)[-1])].contiguous() for n in x}
    g = {n: a.cuda() for n, a in t.items()}
    cq, ck = torch.from_numpy(cuq).cuda(), torch.from_numpy(cuk).cuda()
    o, lse = A.attn_varlen_fwd(g["q"], g["k"], g["v"], cq, dqk ** -0.5, causal, cu_seqlens_k=ck)
    grads = [torch.full_like(g[n], float("nan")) for n in ("q", "k", "v")]
    A.attn_varlen_bwd(g["q"], g["k"], g["v"], o, g["do"], lse, cq, dqk ** -0.5, causal, *grads, cu_seqlens_k=ck)
    torch.cuda.synchronize()
    dq, dk, dvv = (a.float().cpu().numpy() for a in grads)
    for b, (nq, nk) in enumerate(lens):
        sq, sk = slice(int(cuq[b]), int(cuq[b + 1])), slice(int(cuk[b]), int(cuk[b + 1]))
        f = [I.to_f64(t[n][s][None]) for n, s in (("q", sq), ("k", sk), ("v", sk), ("do", sq))]
        rdq, rdk, rdv = oracle.attn_bwd(*f, dqk ** -0.5, causal, q_pos=np.arange(nq) + (nk - nq))
        for what, got, ref in (("dQ", dq[sq], rdq), ("dK", dk[sk], rdk), ("dV", dvv[sk], rdv)):
            assert_close(got[None], ref, f"{what} sequence {b}")


# (d, causal, (queries, keys) of the sequences, element type) at H = 16/8
LARGE = [(128, True, [(513, 513), (1, 300), (1055, 1088), (1100, 1727), (1500, 1500), (2000, 2100)], torch.bfloat16),
         (128, False, [(257, 1000), (1025, 95), (1300, 640)], torch.bfloat16),
         (128, False, [(1025, 95), (257, 1000), (1300, 640)], torch.float16),
         (64, False, [(2561, 8561), (3013, 7900), (2699, 255)], torch.bfloat16),
         (64, False, [(2699, 255), (2561, 7900), (3013, 8561)], torch.float16),
         (64, True, [(8193, 8193), (8400, 8465)], torch.bfloat16)]


@pytest.mark.parametrize("d,causal,lens,dtype", LARGE, ids=["d%d_%s_%s" % (c[0], "c" if c[1] else "nc", c[3]) for c in LARGE])
def test_large_batch_matches_its_sequences_one_by_one(d, causal, lens, dtype):
    """The 64-query dQ kernel and the 256-key dK/dV kernel of d = 64 need many blocks to be chosen: 16 heads of all
    sequences in one call, against one call per sequence, whose few blocks go to the general kernels (themselves
    compared with the oracle elsewhere).  dK and dV are the same bits; dQ differs by the rounding of dP - D, at most
    one ulp of the result plus what one ulp of the row's largest dS moves: that dS is computed here, since a
    sequence of 95 keys has elements of several units and one of a thousand keys none above 0.5."""
    import paper_2603_05451_amd as A
    H, Hkv = 16, 8
    gen = torch.Generator(device="cuda").manual_seed(790 + d)
    mk = lambda n, h: torch.randn(n, h, d, generator=gen, device="cuda").to(dtype)
    tq, tk = (sum(x[i] for x in lens) for i in (0, 1))
    q, k, v, do = mk(tq, H), mk(tk, Hkv), mk(tk, Hkv), mk(tq, H)
    cu = [torch.tensor([0] + list(np.cumsum([x[i] for x in lens])), dtype=torch.int32, device="cuda") for i in (0, 1)]
    o, lse = A.attn_varlen_fwd(q, k, v, cu[0], d ** -0.5, causal, cu_seqlens_k=cu[1])
    grads = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    A.attn_varlen_bwd(q, k, v, o, do, lse, cu[0], d ** -0.5, causal, *grads, cu_seqlens_k=cu[1])
    sq = sk = 0
    for nq, nk in lens:
        a, b = slice(sq, sq + nq), slice(sk, sk + nk)
        one = [torch.tensor([0, n], dtype=torch.int32, device="cuda") for n in (nq, nk)]
        ref = [torch.cat(x, 1) for x in zip(*[A.attn_varlen_bwd(
            q[a, h0:h0 + 2].contiguous(), k[b, h0 // 2:h0 // 2 + 1].contiguous(), v[b, h0 // 2:h0 // 2 + 1].contiguous(),
            o[a, h0:h0 + 2].contiguous(), do[a, h0:h0 + 2].contiguous(), lse[h0:h0 + 2, a].contiguous(), one[0], d ** -0.5,
            causal, cu_seqlens_k=one[1]) for h0 in range(0, H, 2)])]
        torch.cuda.synchronize()
        assert torch.equal(grads[1][b], ref[1]) and torch.equal(grads[2][b], ref[2]), (nq, nk)
        x, y = grads[0][a].float(), ref[0].float()
        for h in range(H):
            move = dq_bound_of_one_ds_ulp(q[a, h], k[b, h // 2], v[b, h // 2], o[a, h], do[a, h], lse[h, a], d ** -0.5, nk - nq, causal)
            assert ((x[:, h] - y[:, h]).abs() <= 2 * half_ulp(dtype) * torch.maximum(x[:, h].abs(), y[:, h].abs()) + move).all(), (nq, nk, h)
        assert ((x - y).norm() / y.norm()).item() < 1e-3
        sq, sk = sq + nq, sk + nk


def test_overlapping_rows_take_the_general_kernels():
    """Inputs whose row stride is shorter than a row (sliding windows over one buffer): results of contiguous
    copies, bit for bit (N a multiple of 128: the same tiles)."""
    import paper_2603_05451_amd as A
    B, N, H, d = 1, 1536, 2, 128
    gen = torch.Generator().manual_seed(781)
    buf = [torch.randn(N * 64 + H * N * 64 + d, generator=gen).bfloat16().cuda() for _ in range(4)]
    q, k, v, do = (t.as_strided((B, N, H, d), (0, 64, N * 64, 1)) for t in buf)
    o, lse = A.attn_fwd_strided(q, k, v, 0.1, True)
    got = A.attn_bwd_strided(q, k, v, o, do, lse, 0.1, True)
    q, k, v, do = (t.contiguous() for t in (q, k, v, do))
    o2, lse2 = A.attn_fwd_strided(q, k, v, 0.1, True)
    ref = A.attn_bwd_strided(q, k, v, o2, do, lse2, 0.1, True)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
