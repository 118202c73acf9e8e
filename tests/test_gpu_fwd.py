"""GPU parity of the forward pass against the CPU fp64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from paper_2603_05451_amd import inputs as I
from parity import (LSE_ABS, assert_close, assert_close_terms, repeated, rounded_reference, same_in_every_repetition,
                    term_magnitudes)

pytestmark = pytest.mark.gpu


def gpu_fwd(w, x):
    import paper_2603_05451_amd as A
    q, k, v = (x[n].cuda() for n in ("q", "k", "v"))
    o, lse = A.attn_fwd(q, k, v, w.scale, w.causal)
    torch.cuda.synchronize()
    return o.float().cpu().numpy(), lse.cpu().numpy()


SMALL = [
    I.CANARY,
    I.Workload("s_d64_c", 2, 4, 2, 384, 64, 64, True, 11),
    I.Workload("s_d64_nc", 1, 3, 1, 256, 64, 64, False, 12),
    I.Workload("s_d96_c", 2, 4, 2, 384, 96, 96, True, 18),
    I.Workload("s_d96_nc", 1, 3, 3, 640, 96, 96, False, 19),
    I.Workload("s_d128_nc", 2, 4, 4, 384, 128, 128, False, 13),
    I.Workload("s_d128_c", 2, 4, 2, 640, 128, 128, True, 14),
    I.Workload("s_d256_c", 1, 4, 2, 384, 256, 256, True, 10),
    I.Workload("s_d256_nc", 2, 2, 2, 256, 256, 256, False, 9),
    I.Workload("s_d192_c", 1, 4, 2, 384, 192, 128, True, 15),
    I.Workload("s_d192_nc", 1, 2, 2, 256, 192, 128, False, 16),
    I.Workload("s_d192_c_outl", 1, 2, 1, 512, 192, 128, True, 17, outlier_frac=0.01),
]


@pytest.mark.parametrize("w", SMALL, ids=lambda w: w.name)
def test_fwd_small_full_parity(oracle, w):
    x = I.make_inputs(w, with_do=False)
    o, lse = gpu_fwd(w, x)
    ro, rlse = oracle.attn_fwd(I.to_f64(x["q"]), I.to_f64(x["k"]), I.to_f64(x["v"]), w.scale, w.causal)
    if w.outlier_frac:
        G = w.H // w.Hkv
        for b in range(w.B):
            for kvh in range(w.Hkv):
                hs = slice(kvh * G, (kvh + 1) * G)
                args = (I.to_f64(x["q"][b, :, hs]), I.to_f64(x["k"][b, :, kvh]), I.to_f64(x["v"][b, :, kvh]),
                        np.zeros((w.N, G, w.dv)), w.scale, w.causal)
                assert_close_terms(o[b, :, hs], ro[b, :, hs], term_magnitudes(*args)[0], f"O {w.name} b{b} kvh{kvh}",
                                   rounded_reference(*args)[0])
    else:
        assert_close(o, ro, f"O {w.name}")
    assert np.abs(lse - rlse).max() <= LSE_ABS, f"LSE {w.name}: {np.abs(lse - rlse).max():.3e}"


FULL = [I.TARGET, I.SWEEP_D64_NC[0], I.SWEEP_D64_NC[5], I.SWEEP_D128_C[0], I.SWEEP_D128_C[4], I.GQA,
        I.MLA_OUTLIER]


@pytest.mark.parametrize("w", FULL, ids=lambda w: w.name)
def test_fwd_full_size_sampled_rows(oracle, w):
    """At the benchmark sizes the oracle computes sampled query rows one by one (all keys)."""
    x = I.make_inputs(w, with_do=False)
    o, lse = gpu_fwd(w, x)
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    rng = np.random.default_rng(w.seed)
    rows = np.unique(np.concatenate([[0, 1, 31, 32, 63, 64, 127, 128, 255, 256, w.N - 257, w.N - 256, w.N - 129, w.N - 128, w.N - 1],
                                     rng.integers(0, w.N, 48)]))
    G = w.H // w.Hkv
    for b, kvh in {(0, 0), (w.B - 1, w.Hkv - 1)}:
        hs = slice(kvh * G, (kvh + 1) * G)
        q = I.to_f64(x["q"][b:b + 1, :, hs][:, rows])
        k = I.to_f64(x["k"][b:b + 1, :, kvh:kvh + 1])
        v = I.to_f64(x["v"][b:b + 1, :, kvh:kvh + 1])
        ro, rlse = oracle.attn_fwd(q, k, v, w.scale, w.causal, q_pos=rows)
        if w.outlier_frac:
            args = (q[0], k[0, :, 0], v[0, :, 0], np.zeros((len(rows), G, w.dv)), w.scale, w.causal)
            assert_close_terms(o[b, :, hs][rows], ro[0], term_magnitudes(*args, q_pos=rows)[0],
                               f"O rows {w.name} b{b} kvh{kvh}", rounded_reference(*args, q_pos=rows)[0])
        else:
            assert_close(o[b:b + 1, :, hs][:, rows], ro, f"O rows {w.name} b{b} kvh{kvh}")
        err = np.abs(lse[b:b + 1, hs][:, :, rows] - rlse).max()
        assert err <= LSE_ABS, f"LSE {w.name}: {err:.3e}"


# (workload, times): the oracle computes the workload's heads, the call runs them `times` over, so that there are enough
# blocks for the kernel with 64 queries per wave (test_dispatch_cpu.py checks that there are)
Q64 = [(I.Workload("q64_nc_2048", 1, 3, 1, 2048, 128, 128, False, 31), 6),
       (I.Workload("q64_nc_2304", 2, 2, 2, 2304, 128, 128, False, 32), 4),
       (I.Workload("q64_c_4096", 1, 4, 2, 4096, 128, 128, True, 37), 6),
       (I.Workload("q64_d64_nc_8192", 1, 2, 1, 8192, 64, 64, False, 33), 3),
       (I.Workload("q64_d64_c_16384", 1, 1, 1, 16384, 64, 64, True, 34), 7),
       (I.Workload("q64_d192_nc_2304", 1, 3, 1, 2304, 192, 128, False, 35), 5),
       (I.Workload("q64_d192_c_8192", 1, 2, 2, 8192, 192, 128, True, 36), 3)]


def repeated_fwd(q, k, v, scale, causal, times):
    """attn_fwd of the heads `times` over; O and LSE of the first repetition, whose bits the others have to have."""
    import paper_2603_05451_amd as A
    o, lse = A.attn_fwd(repeated(q, times), repeated(k, times), repeated(v, times), scale, causal)
    torch.cuda.synchronize()
    H = q.shape[2]
    assert same_in_every_repetition(o, H, 2) and same_in_every_repetition(lse, H, 1)
    return o[:, :, :H].float().cpu().numpy(), lse[:, :H].cpu().numpy()


@pytest.mark.parametrize("w,times", Q64, ids=[w.name for w, _ in Q64])
def test_fwd_64_queries_per_wave_full_parity(oracle, w, times):
    """Shapes that run the kernel with 64 queries per wave (one round of more than 128 blocks, more rounds at longer
    sequences), every row against the oracle: GQA and MHA, key loops of 32 to 256 tiles."""
    x = I.make_inputs(w, with_do=False)
    o, lse = repeated_fwd(x["q"], x["k"], x["v"], w.scale, w.causal, times)
    ro, rlse = oracle.attn_fwd(I.to_f64(x["q"]), I.to_f64(x["k"]), I.to_f64(x["v"]), w.scale, w.causal)
    assert_close(o, ro, f"O {w.name}")
    assert np.abs(lse - rlse).max() <= LSE_ABS, f"LSE {w.name}: {np.abs(lse - rlse).max():.3e}"


# (causal, N, d_qk, d_v, times two heads, element type)
GROWING = [(False, 2048, 128, 128, 9, torch.bfloat16), (True, 8192, 128, 128, 5, torch.bfloat16), (False, 8192, 64, 64, 3, torch.bfloat16),
           (True, 16384, 64, 64, 4, torch.bfloat16), (False, 2048, 192, 128, 9, torch.bfloat16), (True, 8192, 192, 128, 3, torch.bfloat16),
           (False, 2048, 128, 128, 9, torch.float16), (True, 4096, 192, 128, 7, torch.float16)]


@pytest.mark.parametrize("causal,N,d,dv,times,dtype", GROWING, ids=["%s_N%d_d%d_%s" % ("c" if c[0] else "nc", c[1], c[2], c[5]) for c in GROWING])
def test_fwd_growing_scores_restart_with_exact_maxima(oracle, causal, N, d, dv, times, dtype):
    """Scores that grow along the key axis by hundreds of binary orders: relative to the first
    tile's maximum the exponentials overflow, so the pipelined loop of the 64-queries-per-wave
    kernel cannot produce these results; they come from its restart with a row maximum per tile
    and the thresholded rescale (paper Sec. 3.1.4).  Compared on sampled rows."""
    g = torch.Generator("cpu").manual_seed(77)
    H = 2
    q = torch.randn(1, N, H, d, generator=g).abs().to(dtype)
    k = (torch.randn(1, N, 1, d, generator=g).abs() * torch.linspace(0.2, 30.0, N).view(1, N, 1, 1)).to(dtype)
    v = torch.randn(1, N, 1, dv, generator=g).to(dtype)
    scale = d ** -0.5
    o, lse = repeated_fwd(q, k, v, scale, causal, times)
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    rng = np.random.default_rng(5)
    rows = np.unique(np.concatenate([[0, 1, 63, 64, 255, 256, N - 257, N - 1], rng.integers(0, N, 40)]))
    ro, rlse = oracle.attn_fwd(I.to_f64(q[:, rows]), I.to_f64(k), I.to_f64(v), scale, causal, q_pos=rows)
    assert_close(o[:, rows], ro, f"O growing scores causal={causal}")
    err = np.abs(lse[:, :, rows] - rlse).max()
    assert err <= LSE_ABS, f"LSE growing scores: {err:.3e} (values up to {np.abs(rlse).max():.0f})"


STEPS = [(False, 4096, 128, 128, 5), (True, 8192, 192, 128, 3), (False, 8192, 64, 64, 3)]


@pytest.mark.parametrize("causal,N,d,dv,times", STEPS)
def test_fwd_reference_steps_inside_the_pipelined_loop(oracle, causal, N, d, dv, times):
    """Scores that climb along the key axis by about 300 binary orders in small steps: relative to the first
    tile's maximum the tile sums pass 2^90 several times without ever becoming infinite, so the kernel
    with 64 queries per wave must raise its reference inside the pipelined loop (the rescale of paper
    Sec. 3.1.4 with a power-of-two step); no second pass is involved.  Every 37th row against the oracle."""
    g = torch.Generator("cpu").manual_seed(78)
    H = 2
    climb = torch.linspace(0.0, 300.0 / (1.4427 * d ** 0.5), N).view(1, N, 1, 1)         # score = sqrt(d) * climb
    q = (1.0 + 0.1 * torch.randn(1, N, H, d, generator=g)).to(torch.bfloat16)
    k = (climb + 0.1 * torch.randn(1, N, 1, d, generator=g)).to(torch.bfloat16)
    v = torch.randn(1, N, 1, dv, generator=g).to(torch.bfloat16)
    scale = d ** -0.5
    o, lse = repeated_fwd(q, k, v, scale, causal, times)
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    rows = np.unique(np.concatenate([[0, 1, 255, 256, N - 257, N - 1], np.arange(5, N, 37)]))
    ro, rlse = oracle.attn_fwd(I.to_f64(q[:, rows]), I.to_f64(k), I.to_f64(v), scale, causal, q_pos=rows)
    assert_close(o[:, rows], ro, f"O climbing scores causal={causal} d={d}")
    err = np.abs(lse[:, :, rows] - rlse).max()
    assert err <= LSE_ABS * max(1.0, np.abs(rlse).max() / 64), f"LSE climbing scores: {err:.3e} (values up to {np.abs(rlse).max():.0f})"
