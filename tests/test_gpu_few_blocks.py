"""GPU tests of the fixed-length kernels with one wave per SIMD where the number of blocks, not the length, sends a
call to them (more than 128 blocks of 256 rows): short sequences of many heads.  Two heads are generated and
repeated, so that the oracle computes two and every repetition has to reproduce their bits; the scores of the
forward cases grow or climb along the keys, which sends those kernels through the second pass and through the
step of the reference inside the loop."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import LSE_ABS, assert_close

pytestmark = pytest.mark.gpu


def _repeat(t, H):
    return t.repeat(1, 1, H // 2, 1).cuda()


# 144, 384, 140, 448, 136, 224 blocks of 256 queries
FORWARD = [(False, 2048, 18, 128, 128), (True, 4096, 24, 128, 128), (False, 1280, 28, 64, 64), (True, 8192, 14, 64, 64),
           (False, 1024, 34, 192, 128), (True, 4096, 14, 192, 128)]
FORWARD_4_WAVE = [(True, 2048, 26, 128, 128), (True, 8192, 10, 64, 64)]         # one round and a little more under the mask


@pytest.mark.parametrize("causal,N,H,d,dv", FORWARD + FORWARD_4_WAVE)
@pytest.mark.parametrize("kind", ["normal", "growing", "climbing"])
def test_forward(oracle, causal, N, H, d, dv, kind):
    import paper_2603_05451_amd as A
    g = torch.Generator("cpu").manual_seed(300 + d + N)
    q, k, v = (torch.randn(1, N, 2, e, generator=g) for e in (d, d, dv))
    if kind == "growing":        # by hundreds of binary orders: relative to the first tile the exponentials overflow
        q, k = q.abs(), k.abs() * torch.linspace(0.2, 30.0, N).view(1, N, 1, 1)
    if kind == "climbing":       # by 300 binary orders in small steps
        q, k = 1.0 + 0.1 * q, torch.linspace(0.0, 300.0 / (1.4427 * d ** 0.5), N).view(1, N, 1, 1) + 0.1 * k
    q, k, v = (t.bfloat16() for t in (q, k, v))
    o, lse = A.attn_fwd(_repeat(q, H), _repeat(k, H), _repeat(v, H), d ** -0.5, causal)
    torch.cuda.synchronize()
    assert all(torch.equal(o[:, :, h], o[:, :, h % 2]) and torch.equal(lse[:, h], lse[:, h % 2]) for h in range(H))
    rows = np.unique(np.concatenate([[0, 1, 63, 64, 255, 256, N - 257, N - 1], np.arange(5, N, 61)]))
    ro, rlse = oracle.attn_fwd(I.to_f64(q[:, rows]), I.to_f64(k), I.to_f64(v), d ** -0.5, causal, q_pos=rows)
    assert_close(o[:, rows, :2].float().cpu().numpy(), ro, f"O {kind}")
    # (LSE is an fp32 number: half an ulp of one above 1024 is 6e-5, of one above 8192 5e-4)
    assert np.abs(lse[:, :2].cpu().numpy()[:, :, rows] - rlse).max() <= LSE_ABS * max(1.0, np.abs(rlse).max() / 64)


# 328, 136, 136, 416, 448 blocks of 256 queries or keys
BACKWARD = [(True, 1024, 82, 128), (False, 1024, 34, 128), (False, 1024, 34, 64), (True, 4096, 26, 64), (True, 8192, 14, 64)]
BACKWARD_4_WAVE = [(True, 1024, 34, 128), (True, 1024, 50, 64), (True, 2048, 18, 64), (True, 8192, 10, 64)]


@pytest.mark.parametrize("causal,N,H,d", BACKWARD + BACKWARD_4_WAVE)
def test_backward(oracle, causal, N, H, d):
    import paper_2603_05451_amd as A
    x = I.make_inputs(I.Workload("few", 1, 2, 2, N, d, d, causal, 320 + d + H))
    q, k, v, do = (_repeat(x[n], H) for n in ("q", "k", "v", "do"))
    o, lse = A.attn_fwd(q, k, v, d ** -0.5, causal)
    got = A.attn_bwd(q, k, v, o, do, lse, d ** -0.5, causal)
    torch.cuda.synchronize()
    ref = oracle.attn_bwd(*(I.to_f64(x[n]) for n in ("q", "k", "v", "do")), d ** -0.5, causal)
    for what, a, r in zip(("dQ", "dK", "dV"), got, ref):
        assert all(torch.equal(a[:, :, h], a[:, :, h % 2]) for h in range(H)), what
        assert_close(a[:, :, :2].float().cpu().numpy(), r, what)


# heads that do not divide among the 8 XCDs (units of 2, 4 and 8 XCDs, and totals that are not dealt at all), groups of
# unequal width, one tile per head, heads of an XCD's own behind shared ones: the order of the blocks decides which work is done, not what it gives
@pytest.mark.parametrize("B,H,Hkv,N,d,dv", [(1, 12, 4, 512, 128, 128), (1, 2, 1, 1024, 64, 64), (1, 1, 1, 384, 128, 128), (3, 5, 5, 384, 96, 96),
                                            (9, 16, 8, 256, 64, 64), (1, 20, 20, 128, 256, 256), (1, 6, 3, 1024, 192, 128),
                                            (1, 33, 11, 1024, 128, 128), (5, 20, 20, 512, 64, 64), (1, 34, 34, 1024, 64, 64)])
@pytest.mark.parametrize("layout", ["fixed", "views", "packed"])
def test_orders_of_blocks_under_the_mask(oracle, B, H, Hkv, N, d, dv, layout):
    import paper_2603_05451_amd as A
    x = I.make_inputs(I.Workload("order", B, H, Hkv, N, d, dv, True, 340 + B + H))
    q, k, v, do = (x[n].cuda() for n in ("q", "k", "v", "do"))
    if layout == "fixed":
        o, lse = A.attn_fwd(q, k, v, d ** -0.5, True)
        got = (o,) + tuple(A.attn_bwd(q, k, v, o, do, lse, d ** -0.5, True))
    elif layout == "views":
        q, k, v, do = (t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v, do))
        o, lse = A.attn_fwd_strided(q, k, v, d ** -0.5, True)
        got = (o,) + tuple(A.attn_bwd_strided(q, k, v, o, do, lse, d ** -0.5, True))
    else:
        cu = torch.arange(B + 1, dtype=torch.int32, device="cuda") * N
        flat = [t.flatten(0, 1) for t in (q, k, v, do)]
        o, lse = A.attn_varlen_fwd(*flat[:3], cu, d ** -0.5, True)
        got = (o,) + tuple(A.attn_varlen_bwd(*flat[:3], o, flat[3], lse, cu, d ** -0.5, True))
    torch.cuda.synchronize()
    f64 = [I.to_f64(x[n]) for n in ("q", "k", "v", "do")]
    ref = (oracle.attn_fwd(*f64[:3], d ** -0.5, True)[0],) + tuple(oracle.attn_bwd(*f64, d ** -0.5, True))
    for what, a, r in zip(("O", "dQ", "dK", "dV"), got, ref):
        assert_close(a.float().cpu().numpy().reshape(r.shape), r, what)


# blocks that take several key tiles in turns: 257 ... 1536 tiles, totals that are not dealt to the XCDs, a last turn with one
# tile, one query tile group per key tile, pairs of turns under the mask; two query heads per KV head
TURNS = [(False, 128, 258, 1), (False, 128, 264, 2), (False, 384, 86, 1), (False, 256, 260, 1), (True, 128, 512, 1), (True, 256, 256, 2),
         (True, 384, 512, 1)]


@pytest.mark.parametrize("causal,N,Hkv,G", TURNS)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_key_tiles_in_turns(oracle, causal, N, Hkv, G, dtype):
    import paper_2603_05451_amd as A
    x = I.make_inputs(I.Workload("turns", 1, 2 * G, 2, N, 128, 128, causal, 360 + N + Hkv))
    q, do = (x[n].to(dtype).repeat(1, 1, Hkv // 2, 1).cuda() for n in ("q", "do"))
    k, v = (x[n].to(dtype).repeat(1, 1, Hkv // 2, 1).cuda() for n in ("k", "v"))
    o, lse = A.attn_fwd(q, k, v, 128 ** -0.5, causal)
    got = A.attn_bwd(q, k, v, o, do, lse, 128 ** -0.5, causal)
    torch.cuda.synchronize()
    ref = oracle.attn_bwd(*(I.to_f64(x[n].to(dtype)) for n in ("q", "k", "v", "do")), 128 ** -0.5, causal)
    for what, a, r, n in zip(("dQ", "dK", "dV"), got, ref, (2 * G, 2, 2)):
        first = a[:, :, :n]
        assert torch.equal(a, first.repeat(1, 1, Hkv // 2, 1)), what
        assert_close(first.float().cpu().numpy(), r, what)


# the same at d = 64 without a mask: a last turn of 7/8, totals that are not dealt, units of several XCDs, two and three key tiles
# per head, two query heads per KV head
TURNS64 = [(256, 448, 1), (256, 962, 2), (768, 166, 1), (512, 236, 2), (1024, 124, 1)]


@pytest.mark.parametrize("N,Hkv,G", TURNS64)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_key_tiles_in_turns_d64(oracle, N, Hkv, G, dtype):
    import paper_2603_05451_amd as A
    x = I.make_inputs(I.Workload("turns", 1, 2 * G, 2, N, 64, 64, False, 380 + N + Hkv))
    q, do = (x[n].to(dtype).repeat(1, 1, Hkv // 2, 1).cuda() for n in ("q", "do"))
    k, v = (x[n].to(dtype).repeat(1, 1, Hkv // 2, 1).cuda() for n in ("k", "v"))
    o, lse = A.attn_fwd(q, k, v, 0.125, False)
    got = A.attn_bwd(q, k, v, o, do, lse, 0.125, False)
    torch.cuda.synchronize()
    ref = oracle.attn_bwd(*(I.to_f64(x[n].to(dtype)) for n in ("q", "k", "v", "do")), 0.125, False)
    for what, a, r, n in zip(("dQ", "dK", "dV"), got, ref, (2 * G, 2, 2)):
        first = a[:, :, :n]
        assert torch.equal(a, first.repeat(1, 1, Hkv // 2, 1)), what
        assert_close(first.float().cpu().numpy(), r, what)
