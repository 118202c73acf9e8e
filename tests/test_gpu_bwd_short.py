"""GPU tests of the backward kernel that holds all keys of a sequence in one block (bwd_short in csrc/dispatch.h): edges of its 32-key blocks,
32-query tiles and sizes of block, more and fewer queries than keys, heads per KV head, layouts, both types, against the oracle.  Two KV
heads are generated and repeated where the rule asks for many: the oracle computes two and every repetition has to reproduce their bits."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import assert_close

pytestmark = pytest.mark.gpu

# d, queries, keys, query heads per KV head, KV heads, causal, layout
CASES = [
    (64, 33, 33, 1, 2, True, "bhnd"), (64, 100, 127, 1, 2, False, "room"), (64, 128, 128, 1, 2, True, "fixed"), (64, 129, 129, 2, 512, True, "qkv"),
    (64, 255, 255, 1, 320, False, "room"), (64, 256, 256, 2, 320, True, "fixed"), (64, 7, 257, 3, 2, True, "bhnd"), (64, 257, 257, 1, 200, True, "qkv"),
    (64, 300, 511, 1, 200, False, "bhnd"), (64, 512, 512, 1, 240, True, "fixed"), (64, 700, 200, 1, 512, False, "room"), (64, 64, 512, 1, 2, True, "room"),
    (96, 40, 97, 1, 2, True, "bhnd"), (96, 128, 128, 1, 2, False, "fixed"), (96, 161, 161, 2, 512, True, "room"), (96, 256, 256, 1, 512, False, "fixed"),
    (96, 99, 99, 1, 2, False, "qkv"), (96, 70, 250, 1, 2, False, "bhnd"),
    (128, 50, 50, 1, 2, True, "room"), (128, 128, 128, 1, 2, True, "fixed"), (128, 65, 128, 3, 512, False, "bhnd"), (128, 129, 129, 1, 512, True, "qkv"),
    (128, 200, 256, 2, 256, True, "bhnd"), (128, 256, 256, 1, 256, False, "fixed"), (128, 400, 225, 1, 512, False, "room"),
]


def _inputs(d, Nq, Nk, G, Hkv, layout, dtype, seed):
    """q, k, v, do as [1, N, heads, d] views of the layout; the two distinct KV heads (and their query heads) on the CPU."""
    g = torch.Generator("cpu").manual_seed(seed)
    two = [torch.randn(1, n, h, d, generator=g).to(dtype) for n, h in ((Nq, 2 * G), (Nk, 2), (Nk, 2), (Nq, 2 * G))]
    out = [t.repeat(1, 1, Hkv // 2, 1).cuda() for t in two]
    if layout == "bhnd":
        out = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in out]
    if layout == "qkv":
        f = torch.cat(out[:3], dim=2)
        out[:3] = f[:, :, :G * Hkv], f[:, :, G * Hkv:(G + 1) * Hkv], f[:, :, (G + 1) * Hkv:]
    if layout == "room":                # rows behind the last one hold NaN
        wide = [torch.full((1, t.shape[1] + 40, *t.shape[2:]), float("nan"), dtype=dtype, device="cuda") for t in out]
        for w, t in zip(wide, out):
            w[:, :t.shape[1]] = t
        out = [w[:, :t.shape[1]] for w, t in zip(wide, out)]
    return two, out


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("d,Nq,Nk,G,Hkv,causal,layout", CASES)
def test_against_the_oracle(oracle, d, Nq, Nk, G, Hkv, causal, layout, dtype):
    import paper_2603_05451_amd as A
    two, (q, k, v, do) = _inputs(d, Nq, Nk, G, Hkv, layout, dtype, 900 + d + Nq + Nk)
    scale = d ** -0.5
    if layout == "fixed":
        o, lse = A.attn_fwd(q, k, v, scale, causal)
        got = A.attn_bwd(q, k, v, o, do, lse, scale, causal)
        again = A.attn_bwd_strided(q, k, v, o, do, lse, scale, causal)
    else:
        o, lse = A.attn_fwd_strided(q, k, v, scale, causal)
        # gradients into buffers with room behind the last row, which stays as it is
        wide = [torch.full((1, t.shape[1] + 3, *t.shape[2:]), 7.0, dtype=dtype, device="cuda") for t in (q, k, v)]
        got = A.attn_bwd_strided(q, k, v, o, do, lse, scale, causal, *(w[:, :t.shape[1]] for w, t in zip(wide, (q, k, v))))
        again = A.attn_bwd_strided(*(t.contiguous() for t in (q, k, v, o, do)), lse, scale, causal)
        torch.cuda.synchronize()
        assert all((w[:, t.shape[1]:] == 7.0).all() for w, t in zip(wide, (q, k, v)))
    torch.cuda.synchronize()
    ref = oracle.attn_bwd(*(I.to_f64(t) for t in two), scale, causal, q_pos=np.arange(Nq) + Nk - Nq if causal else None)
    for what, a, b, r, heads in zip(("dQ", "dK", "dV"), got, again, ref, (2 * G, 2, 2)):
        assert torch.equal(a, b), what                                          # no layout changes a bit, nor does a second call
        assert torch.equal(a, a[:, :, :heads].repeat(1, 1, Hkv // 2, 1)), what
        assert_close(a[:, :, :heads].float().cpu().numpy(), r, f"{what} d{d} {Nq}x{Nk}")


@pytest.mark.parametrize("d", [64, 96, 128])
def test_one_key(d):
    """P = 1 and dS = 0: dQ = dK = 0 but for rounding (1e-5), dV the dO of the query."""
    import paper_2603_05451_amd as A
    _, (q, k, v, do) = _inputs(d, 1, 1, 1, 2, "bhnd", torch.bfloat16, 950)
    o, lse = A.attn_fwd_strided(q, k, v, d ** -0.5, True)
    dq, dk, dv = A.attn_bwd_strided(q, k, v, o, do, lse, d ** -0.5, True)
    torch.cuda.synchronize()
    assert dq.float().abs().max() <= 1e-5 and dk.float().abs().max() <= 1e-5 and torch.equal(dv, do)


PASSES = [(64, 128, 2, False), (64, 256, 64, True), (128, 128, 2, True), (128, 256, 64, False), (96, 128, 2, False)]


@pytest.mark.parametrize("d,N,B,causal", PASSES)
def test_passes_compose(d, N, B, causal):
    """The calls for single passes give the bits of the whole one, in every order, whatever the workspace holds."""
    import paper_2603_05451_amd as A
    g = torch.Generator(device="cuda").manual_seed(960 + d)
    q, k, v, do = (torch.randn(B, N, 8, d, generator=g, device="cuda").bfloat16() for _ in range(4))
    o, lse = A.attn_fwd(q, k, v, d ** -0.5, causal)
    ref = A.attn_bwd(q, k, v, o, do, lse, d ** -0.5, causal)
    for order in ((1, 2, 4), (4, 2), (2, 4), (3, 4)):
        got = [torch.full_like(t, float("nan")) for t in (q, k, v)]
        ws = torch.full((A.attn_bwd_workspace_bytes(B, 8, 8, N, d, d),), 0xFF, dtype=torch.uint8, device="cuda")
        for p in order:
            A.attn_bwd(q, k, v, o, do, lse, d ** -0.5, causal, *got, ws, phases=p)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, ref)), order


@pytest.mark.parametrize("d,N,B,causal", PASSES)
def test_one_pass_launches_one_kernel(d, N, B, causal):
    """The workspace is neither read nor written but by the prepare pass, and a call for one pass writes that pass's results alone."""
    import paper_2603_05451_amd as A
    g = torch.Generator(device="cuda").manual_seed(965 + d)
    q, k, v, do = (torch.randn(B, N, 8, d, generator=g, device="cuda").bfloat16() for _ in range(4))
    o, lse = A.attn_fwd(q, k, v, d ** -0.5, causal)
    for phases in range(1, 8):
        got = [torch.full_like(t, 7.0) for t in (q, k, v)]
        ws = torch.full((A.attn_bwd_workspace_bytes(B, 8, 8, N, d, d),), 0xA5, dtype=torch.uint8, device="cuda")
        A.attn_bwd(q, k, v, o, do, lse, d ** -0.5, causal, *got, ws, phases=phases)
        torch.cuda.synchronize()
        assert bool((ws == 0xA5).all()) == (phases not in (1, 3)), phases
        assert [bool((t == 7.0).all()) for t in got] == [not phases & 4, not phases & 2, not phases & 2], phases


@pytest.mark.parametrize("d,N,Hkv,row", [(64, 128, 256, 40), (64, 256, 320, 70), (64, 512, 240, 300), (96, 250, 160, 133), (128, 128, 224, 5), (128, 256, 160, 200)])
def test_a_query_that_is_no_number(d, N, Hkv, row):
    """Under the mask it reaches the dV of the keys that it sees and of no other."""
    import paper_2603_05451_amd as A
    _, (q, k, v, do) = _inputs(d, N, N, 1, Hkv, "bhnd", torch.bfloat16, 990 + d)
    o, lse = A.attn_fwd_strided(q, k, v, d ** -0.5, True)
    clean = A.attn_bwd_strided(q, k, v, o, do, lse, d ** -0.5, True)[2]
    q[:, row] = float("nan")
    o, lse = A.attn_fwd_strided(q, k, v, d ** -0.5, True)
    dv = A.attn_bwd_strided(q, k, v, o, do, lse, d ** -0.5, True)[2]
    torch.cuda.synchronize()
    assert torch.isnan(dv[:, :row + 1].float()).all() and torch.equal(dv[:, row + 1:], clean[:, row + 1:])


@pytest.mark.parametrize("d,Nq,Nk,causal", [(64, 33, 40, True), (64, 70, 200, False), (64, 90, 300, True), (64, 50, 512, False), (96, 33, 97, False), (96, 100, 200, True),
                                            (128, 50, 100, True), (128, 97, 250, False)])
def test_a_key_that_nobody_sees(d, Nq, Nk, causal):
    """A row of K whose scores are all -inf has P = 0 everywhere, in the rows past the end of the last query tile, too: dK = dV = 0 there, and
    the other keys' gradients are those of the same keys with a row of finite scores so low that P = 0."""
    import paper_2603_05451_amd as A
    _, (q, k, v, do) = _inputs(d, Nq, Nk, 1, 2, "room", torch.bfloat16, 995 + d)
    q = q.abs() + 0.5
    got = []
    for low in (-1e4, float("-inf")):
        k[:, 5] = low
        o, lse = A.attn_fwd_strided(q, k, v, d ** -0.5, causal)
        got.append(A.attn_bwd_strided(q, k, v, o, do, lse, d ** -0.5, causal)[1:])
    torch.cuda.synchronize()
    for what, a, b in zip(("dK", "dV"), *got):
        assert torch.isfinite(b.float()).all() and (b[:, 5] == 0).all() and torch.equal(a, b), what
