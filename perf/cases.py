"""The calls that the speed of this library is measured on: attention as training, prefill and decoding
use it, through the public entry points of the Python binding.

A case is a dict of plain values.  Its "kind" says which calls one pass makes:

  train    attn_fwd + attn_bwd            [B, N, H, d] batches, N a multiple of 128: a training step's attention
  prefill  attn_fwd                       the same layout, forward only: a prompt
  packed   attn_varlen_fwd + _bwd         sequences of mixed lengths packed back to back: a padding-free training batch
  views    attn_fwd_strided + _bwd        any N, in the layouts models hold: "qkv" = slices of one fused projection,
                                          "bhnd" = [B, H, N, d] storage
  chunk    attn_fwd_strided               Nq new tokens per sequence against a KV cache that already holds Nk (chunked
                                          prefill, speculative decoding; Nq = 1 is a decode step)
  paged    attn_varlen_fwd                one query per sequence against packed caches of mixed lengths: a decode step
                                          of a serving batch
"""
import math
import random

import torch

import paper_2603_05451_amd as A

DIMS = [(64, 64), (96, 96), (128, 128), (192, 128), (256, 256)]


def _case(name, kind, B, H, Hkv, Nq, Nk, dqk, dv, causal, dtype="bf16", layout="", lo=0, hi=0, len_seed=0):
    return {"name": name, "kind": kind, "B": B, "H": H, "Hkv": Hkv, "Nq": Nq, "Nk": Nk, "dqk": dqk, "dv": dv,
            "causal": causal, "dtype": dtype, "layout": layout, "lo": lo, "hi": hi, "len_seed": len_seed}


def listed():
    return [
        # the smallest training call the repository names (its canary): nothing but launches and call overhead
        _case("train_tiny", "train", 1, 2, 2, 128, 128, 64, 64, False),
        # short sequences of an encoder, the head of the 16 384-token sweep at d = 64 without a mask
        _case("train_d64_N512", "train", 32, 16, 16, 512, 512, 64, 64, False),
        # a decoder's training step on short contexts, from the causal sweep at d = 128
        _case("train_d128_causal_N1024", "train", 16, 16, 16, 1024, 1024, 128, 128, True),
        # the benchmark's shape: long sequences, no mask
        _case("train_d128_N8192", "train", 2, 16, 16, 8192, 8192, 128, 128, False),
        # prompt of a grouped-query model (the GQA workload, forward only)
        _case("prefill_gqa_N8192", "prefill", 2, 32, 8, 8192, 8192, 128, 128, True),
        # latent-attention head dims in training, at a usual context length
        _case("train_d192x128_causal_N4096", "train", 1, 16, 16, 4096, 4096, 192, 128, True),
        # the largest head dim in training (hidden 2048, as the d = 256 workload)
        _case("train_d256_causal_N2048", "train", 4, 8, 8, 2048, 2048, 256, 256, True),
        # padding-free training batch of a grouped-query model: 16 sequences, 64 ... 8192 tokens
        _case("packed_gqa_d128", "packed", 16, 32, 8, 0, 0, 128, 128, True, lo=64, hi=8192, len_seed=8),
        # fp16 encoder whose tensors are [B, H, N, d] and whose length is no multiple of a tile
        _case("views_bhnd_d64_fp16_N1000", "views", 8, 12, 12, 1000, 1000, 64, 64, False, "fp16", "bhnd"),
        # chunked prefill: 512 new tokens of one request against the 8 k tokens already in the cache
        _case("chunk_512_of_8192", "chunk", 1, 32, 8, 512, 8192, 128, 128, True),
        # one decode step of 32 requests, equal lengths, against a [B, Nmax, Hkv, d] cache
        _case("decode_B32_N4001", "chunk", 32, 32, 8, 1, 4001, 128, 128, True),
        # one decode step of a serving batch whose requests are at different lengths
        _case("decode_mixed_B48", "paged", 48, 32, 8, 1, 0, 128, 128, True, lo=64, hi=8192, len_seed=12),
    ]


def _lengths(case):
    """Log-uniform sequence lengths in [lo, hi], in drawn order."""
    r = random.Random(case["len_seed"])
    return [int(round(math.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]))))) for _ in range(case["B"])]


def _sequences(case):
    """(queries, keys) of every sequence of a pass."""
    if case["kind"] == "packed":
        return [(n, n) for n in _lengths(case)]
    if case["kind"] == "paged":
        return [(1, n) for n in _lengths(case)]
    return [(case["Nq"], case["Nk"])] * case["B"]


def _backward(case):
    return case["kind"] in ("train", "packed", "views")


def work(case):
    H, Hkv, dqk, dv = case["H"], case["Hkv"], case["dqk"], case["dv"]
    seqs = _sequences(case)
    pairs = sum(nq * nk - (nq * (nq - 1) // 2 if case["causal"] else 0) for nq, nk in seqs)
    tq, tk = sum(s[0] for s in seqs), sum(s[1] for s in seqs)
    q, o, kv, lse = tq * H * dqk * 2, tq * H * dv * 2, tk * Hkv * (dqk + dv) * 2, tq * H * 4
    flops = 2 * pairs * H * (dqk + dv)                     # S = Q K^T and O = P V
    nbytes = q + kv + o + lse
    if _backward(case):
        flops += 2 * pairs * H * (3 * dqk + 2 * dv)        # S again, dP, dV, dK, dQ
        nbytes += q + kv + 2 * o + lse + q + kv            # q, k, v, o, d_o, lse in; dq, dk, dv out
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Against 64 bits the outputs are off by 2.0e-3 ... 2.5e-3 in bf16 (rounding of O, P and dS to 8
    # bits) and by 3e-4 in fp16 (11 bits): about four times that.
    return {"rel": 1.2e-3 if case["dtype"] == "fp16" else 1e-2}


def draw(rng):
    """One more case: the kinds in the listed ones' proportion, sizes spread over their logarithm."""
    top = max((work(c) for c in listed()), key=lambda w: w["flops"])["flops"]
    logu = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        kind = rng.choice(["train", "train", "train", "prefill", "packed", "packed", "views", "views",
                           "chunk", "chunk", "chunk", "paged", "paged"])
        dqk, dv = rng.choice([(64, 64), (128, 128), (128, 128)] + DIMS)
        Hkv = rng.choice([1, 2, 4, 8, 8, 12, 16])
        H = Hkv * rng.choice([1, 1, 2, 4, 8])
        if H > 64:
            continue
        causal = rng.random() < 0.6
        dtype = "fp16" if rng.random() < 0.25 else "bf16"
        if kind in ("train", "prefill"):
            N = 128 * logu(1, 64)
            c = _case("", kind, logu(1, 32), H, Hkv, N, N, dqk, dv, causal, dtype)
        elif kind == "views":
            N = logu(16, 8192)
            c = _case("", kind, logu(1, 32), H, Hkv, N, N, dqk, dv, causal, dtype, rng.choice(["qkv", "bhnd"]))
        elif kind == "packed":
            c = _case("", kind, logu(2, 64), H, Hkv, 0, 0, dqk, dv, causal, dtype, lo=logu(16, 256), hi=logu(512, 8192),
                      len_seed=rng.randrange(1 << 20))
        elif kind == "chunk":
            Nq = 1 if rng.random() < 0.5 else logu(2, 1024)
            c = _case("", kind, logu(1, 64), H, Hkv, Nq, max(Nq, logu(64, 32768)), dqk, dv, True, dtype)
        else:
            c = _case("", kind, logu(2, 128), H, Hkv, 1, 0, dqk, dv, True, dtype, lo=logu(16, 512), hi=logu(1024, 16384),
                      len_seed=rng.randrange(1 << 20))
        w = work(c)
        if w["flops"] <= 0.6 * top and w["bytes"] <= 1.5e9:      # the dearest head dims run at half the rate
            del c["name"]
            return c


def prepare(case, seed):
    B, H, Hkv, Nq, Nk, dqk, dv = (case[n] for n in ("B", "H", "Hkv", "Nq", "Nk", "dqk", "dv"))
    dtype = torch.float16 if case["dtype"] == "fp16" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, dtype=torch.float32, device="cuda").to(dtype)

    s = {"kind": case["kind"], "scale": dqk ** -0.5, "causal": case["causal"]}
    if case["kind"] in ("train", "prefill"):
        s["q"], s["k"], s["v"] = normal(B, Nq, H, dqk), normal(B, Nk, Hkv, dqk), normal(B, Nk, Hkv, dv)
        if case["kind"] == "train":
            s["do"] = normal(B, Nq, H, dv)
    elif case["kind"] in ("packed", "paged"):
        seqs = _sequences(case)
        cu = lambda lens: torch.tensor([sum(lens[:i]) for i in range(B + 1)], dtype=torch.int32, device="cuda")
        tq, tk = sum(x[0] for x in seqs), sum(x[1] for x in seqs)
        s["q"], s["k"], s["v"] = normal(tq, H, dqk), normal(tk, Hkv, dqk), normal(tk, Hkv, dv)
        s["cu_q"], s["cu_k"] = cu([x[0] for x in seqs]), cu([x[1] for x in seqs])
        if case["kind"] == "packed":
            s["do"] = normal(tq, H, dv)
        else:                                              # a decode loop keeps its output buffers and its workspace
            s["o"] = torch.empty(tq, H, dv, dtype=dtype, device="cuda")
            s["lse"] = torch.empty(H, tq, dtype=torch.float32, device="cuda")
            s["ws"] = torch.empty(A.attn_varlen_workspace_bytes(B, tq, tk, H, Hkv, dqk, dv, False), dtype=torch.uint8,
                                  device="cuda")
    elif case["kind"] == "views":
        s["layout"] = case["layout"]
        if case["layout"] == "qkv" and dqk == dv:
            qkv = normal(B, Nq, H + 2 * Hkv, dqk)
            s["q"], s["k"], s["v"] = qkv[:, :, :H], qkv[:, :, H:H + Hkv], qkv[:, :, H + Hkv:]
            s["do"] = normal(B, Nq, H, dv)
        else:
            s["layout"] = "bhnd"
            s["q"], s["k"], s["v"], s["do"] = (normal(B, h, Nq, d).transpose(1, 2)
                                               for h, d in ((H, dqk), (Hkv, dqk), (Hkv, dv), (H, dv)))
    else:                                                  # chunk: views of a cache with room for more tokens
        room = (Nk + 255) // 256 * 256
        s["q"] = normal(B, Nq, H, dqk)
        s["k"], s["v"] = normal(B, room, Hkv, dqk)[:, :Nk], normal(B, room, Hkv, dv)[:, :Nk]
        s["o"] = torch.empty(B, Nq, H, dv, dtype=dtype, device="cuda")
        s["lse"] = torch.empty(B, H, Nq, dtype=torch.float32, device="cuda")
        s["ws"] = torch.empty(A.attn_strided_workspace_bytes(B, H, Hkv, Nq, Nk, dqk, dv, False), dtype=torch.uint8,
                              device="cuda")
    return s


def run(s):
    kind, q, k, v, scale, causal = s["kind"], s["q"], s["k"], s["v"], s["scale"], s["causal"]
    if kind == "train":
        o, lse = A.attn_fwd(q, k, v, scale, causal)
        return (o, lse) + A.attn_bwd(q, k, v, o, s["do"], lse, scale, causal)
    if kind == "prefill":
        return A.attn_fwd(q, k, v, scale, causal)
    if kind == "packed":
        o, lse = A.attn_varlen_fwd(q, k, v, s["cu_q"], scale, causal)
        return (o, lse) + A.attn_varlen_bwd(q, k, v, o, s["do"], lse, s["cu_q"], scale, causal)
    if kind == "views":
        if s["layout"] == "qkv":
            H, Hkv = q.shape[2], k.shape[2]
            o, lse = A.attn_fwd_strided(q, k, v, scale, causal)
            dqkv = torch.empty(q.shape[0], q.shape[1], H + 2 * Hkv, q.shape[3], dtype=q.dtype, device=q.device)
            A.attn_bwd_strided(q, k, v, o, s["do"], lse, scale, causal,
                               dq=dqkv[:, :, :H], dk=dqkv[:, :, H:H + Hkv], dv=dqkv[:, :, H + Hkv:])
            return o, lse, dqkv
        like = lambda t: torch.empty_like(t.transpose(1, 2)).transpose(1, 2)       # [B, heads, N, d] storage again
        o = torch.empty(q.shape[0], q.shape[2], q.shape[1], v.shape[3], dtype=q.dtype, device=q.device).transpose(1, 2)
        o, lse = A.attn_fwd_strided(q, k, v, scale, causal, o=o)
        dq, dk, dv = A.attn_bwd_strided(q, k, v, o, s["do"], lse, scale, causal, dq=like(q), dk=like(k), dv=like(v))
        return o, lse, dq, dk, dv
    if kind == "chunk":
        return A.attn_fwd_strided(q, k, v, scale, causal, o=s["o"], lse=s["lse"], workspace=s["ws"])
    return A.attn_varlen_fwd(q, k, v, s["cu_q"], scale, causal, o=s["o"], lse=s["lse"], workspace=s["ws"],
                             cu_seqlens_k=s["cu_k"])


def _exact_sequence(q, k, v, do, scale, causal):
    """Attention of one sequence in 64 bits: q [n, H, d], k [m, Hkv, d], v [m, Hkv, dv] -> o, lse [H, n] and, with
    do, dq, dk, dv.  The last query is aligned with the last key."""
    n, H, _ = q.shape
    m, Hkv, _ = k.shape
    o = torch.empty(n, H, v.shape[2], dtype=torch.float64, device=q.device)
    lse = torch.empty(H, n, dtype=torch.float64, device=q.device)
    if do is not None:
        dq, dk, dv = (torch.zeros(t.shape, dtype=torch.float64, device=q.device) for t in (q, k, v))
    hidden = None
    if causal:
        hidden = torch.arange(m, device=q.device)[None, :] > torch.arange(n, device=q.device)[:, None] + (m - n)
    for h in range(H):
        g = h // (H // Hkv)
        qh, kh, vh = q[:, h].double(), k[:, g].double(), v[:, g].double()
        p = qh @ kh.T * scale
        if hidden is not None:
            p.masked_fill_(hidden, -math.inf)
        lse[h] = torch.logsumexp(p, dim=1)
        p.sub_(lse[h][:, None]).exp_()
        o[:, h] = p @ vh
        if do is not None:
            doh = do[:, h].double()
            dv[:, g] += p.T @ doh
            ds = (doh @ vh.T).sub_((doh * o[:, h]).sum(1, keepdim=True)).mul_(p).mul_(scale)
            dq[:, h] = ds @ kh
            dk[:, g] += ds.T @ qh
    return (o, lse) if do is None else (o, lse, dq, dk, dv)


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] in ("packed", "paged"):
        cq = s["cu_q"].tolist()
        ck = cq if case["kind"] == "packed" else s["cu_k"].tolist()
        parts = [_exact_sequence(s["q"][cq[b]:cq[b + 1]], s["k"][ck[b]:ck[b + 1]], s["v"][ck[b]:ck[b + 1]],
                                 s["do"][cq[b]:cq[b + 1]] if "do" in s else None, s["scale"], case["causal"])
                 for b in range(case["B"])]
        return tuple(torch.cat(x, dim=1 if i == 1 else 0) for i, x in enumerate(zip(*parts)))      # lse is [H, T]
    parts = [_exact_sequence(s["q"][b], s["k"][b], s["v"][b], s["do"][b] if "do" in s else None, s["scale"], case["causal"])
             for b in range(case["B"])]
    out = tuple(torch.stack(x) for x in zip(*parts))
    if s.get("layout") == "qkv":
        return out[0], out[1], torch.cat(out[2:], dim=2)
    return out
