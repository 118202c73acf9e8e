"""GPU tests of the d = 64 backward kernels with three blocks per CU (lean_blocks in csrc/dispatch.h): ragged and whole tiles, more keys than
queries, packed sequences with and without rows, both types.  Two KV heads are generated and repeated until the rule asks for the lean kernels:
every repetition gives the bits of the call with two heads, which runs the wide ones, and the two are checked against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import assert_close
from test_gpu_bwd_short import _inputs

pytestmark = pytest.mark.gpu

# queries, keys, query heads per KV head, KV heads, causal, layout
CASES = [(640, 640, 1, 104, False, "fixed"), (640, 640, 2, 130, True, "fixed"), (515, 515, 1, 130, False, "room"), (515, 515, 1, 130, True, "room"),
         (577, 577, 2, 130, True, "qkv"), (130, 700, 1, 110, True, "bhnd"), (159, 700, 3, 90, False, "bhnd"), (600, 513, 1, 130, False, "room")]
PACKED = [0, 1, 131, 131, 195, 895, 1228, 1900]           # ends of the sequences, one of them empty


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("Nq,Nk,G,Hkv,causal,layout", CASES)
def test_the_bits_of_the_wide_kernels(oracle, Nq, Nk, G, Hkv, causal, layout, dtype):
    import paper_2603_05451_amd as A
    fwd, bwd = (A.attn_fwd, A.attn_bwd) if layout == "fixed" else (A.attn_fwd_strided, A.attn_bwd_strided)
    two, few = _inputs(64, Nq, Nk, G, 2, layout, dtype, 970 + Nq + Nk)
    _, many = _inputs(64, Nq, Nk, G, Hkv, layout, dtype, 970 + Nq + Nk)
    got = []
    for q, k, v, do in (few, many):
        o, lse = fwd(q, k, v, 0.125, causal)
        got.append(bwd(q, k, v, o, do, lse, 0.125, causal))
    torch.cuda.synchronize()
    ref = oracle.attn_bwd(*(I.to_f64(t) for t in two), 0.125, causal, q_pos=np.arange(Nq) + Nk - Nq if causal else None)
    for what, a, b, r in zip(("dQ", "dK", "dV"), *got, ref):
        assert torch.equal(a.repeat(1, 1, Hkv // 2, 1), b), what
        assert_close(a.float().cpu().numpy(), r, f"{what} {Nq}x{Nk}")


@pytest.mark.parametrize("causal", [False, True])
def test_packed_sequences(causal):
    import paper_2603_05451_amd as A
    g = torch.Generator("cpu").manual_seed(980)
    cu = torch.tensor(PACKED, dtype=torch.int32, device="cuda")
    base = [torch.randn(PACKED[-1], 2, 64, generator=g).bfloat16().cuda() for _ in range(4)]
    got = []
    for times in (1, 30):
        q, k, v, do = (t.repeat(1, times, 1) for t in base)
        o, lse = A.attn_varlen_fwd(q, k, v, cu, 0.125, causal)
        got.append(A.attn_varlen_bwd(q, k, v, o, do, lse, cu, 0.125, causal))
    torch.cuda.synchronize()
    for what, a, b in zip(("dQ", "dK", "dV"), *got):
        assert torch.isfinite(a.float()).all() and torch.equal(a.repeat(1, 30, 1), b), what
