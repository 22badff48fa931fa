"""Performance cases of the S2-Attn layer: what a training step, an evaluation forward or a
prefill asks of the library, called through paper_2309_12307_amd.binding.

A case is a dict of plain values:
  dtype           "bf16" or "f32" (type of q, k, v, o and the gradients; lse is fp32)
  B N H Hkv D G   batch, tokens, query heads, kv heads, head dimension, group size
  passes          "fwd_bwd" (training step of the layer) or "fwd" (evaluation, prefill)
  call            how the program calls the library:
    "tensors"     s2attn_fwd / s2attn_bwd on contiguous tensors, published defaults
    "full"        no head shifts; with G == N this is plain causal attention
    "variant2"    the wrap-around group is cut at its seam; q, k, v and their gradients are
                  views of one packed projection tensor
    "shard"       heads [offset, offset + H) of a layer of heads_total heads (tensor parallel)
    "static"      backward on the library's own scratch, no workspace
    "shift"       a shift other than G / 2, on the second half of the heads
"""
import math

import torch

from paper_2309_12307_amd import binding

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, dtype, B, N, H, Hkv, D, G, passes="fwd_bwd", call="tensors", shift=-1, heads_total=0, offset=0):
    c = dict(dtype=dtype, B=B, N=N, H=H, Hkv=Hkv, D=D, G=G, passes=passes, call=call, shift=shift,
             heads_total=heads_total, offset=offset)
    return dict(c, name=name) if name else c


def listed():
    return [
        # fp32 configuration of the repository: the smallest call, all latency
        _case("fp32_256", "f32", 1, 256, 4, 4, 64, 64),
        # the same mode at a size where a numerical check of a model layer is run
        _case("fp32_4k", "f32", 1, 4096, 8, 8, 128, 1024),
        # smallest bf16 step with grouped heads, backward on the library's scratch (graph capture)
        _case("train_1k_static", "bf16", 1, 1024, 4, 2, 128, 256, call="static"),
        # short context, batch of two, packed qkv projection, seam of the wrap group cut
        _case("train_4k_packed_variant2", "bf16", 2, 4096, 32, 8, 128, 1024, call="variant2"),
        # 7B-shaped layer at the method's shortest context (8192 tokens, groups of 2048)
        _case("train_8k_mha", "bf16", 1, 8192, 32, 32, 128, 2048),
        # one kv head for all query heads: it serves shifted and unshifted heads
        _case("train_8k_mqa", "bf16", 1, 8192, 32, 1, 128, 2048),
        # one tensor-parallel rank: 8 of 32 heads, four of them shifted
        _case("train_16k_shard", "bf16", 1, 16384, 8, 8, 128, 4096, call="shard", heads_total=32, offset=12),
        # 64-wide heads at 32k
        _case("train_32k_d64", "bf16", 1, 32768, 32, 32, 64, 8192),
        # 7B-shaped layer at 32k: the headline workload
        _case("train_32k_mha", "bf16", 1, 32768, 32, 32, 128, 8192),
        # 70B-shaped layer at 32k, 8 query heads per kv head
        _case("train_32k_gqa", "bf16", 1, 32768, 64, 8, 128, 8192),
        # inference keeps full attention: prefill of 32k tokens
        _case("prefill_32k_full", "bf16", 1, 32768, 32, 32, 128, 32768, passes="fwd", call="full"),
        # the longest context of the paper: 100 000 tokens, a group size that no tile divides
        _case("train_100k", "bf16", 1, 100000, 32, 32, 128, 25000),
    ]


def _pairs(c):
    """(query, key) pairs that attend: causal inside every group (or part of a cut group)."""
    G, NG = c["G"], c["N"] // c["G"]
    whole = G * (G + 1) // 2
    total = c["H"] * NG * whole
    if c["call"] == "variant2":
        a = G - G // 2
        total -= (c["H"] // 2) * (whole - a * (a + 1) // 2 - (G - a) * (G - a + 1) // 2)
    return c["B"] * total


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    q = case["B"] * case["N"] * case["H"] * case["D"] * e
    kv = case["B"] * case["N"] * case["Hkv"] * case["D"] * e
    lse = case["B"] * case["N"] * case["H"] * 4
    # forward: 4 D per pair (two products); backward: 10 D (five products)
    if case["passes"] == "fwd":
        return {"bytes": 2 * q + 2 * kv + lse, "flops": 4.0 * case["D"] * _pairs(case)}
    return {"bytes": 4 * q + 4 * kv + lse, "flops": 14.0 * case["D"] * _pairs(case)}


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(x, multiple):
    """x as a positive multiple of `multiple`, or just even where multiple is 0."""
    m = multiple or 2
    return max(m, x // m * m)


def _draw(rng):
    fp32 = rng.random() < 0.2
    if fp32:
        D = rng.choice([64, 128])
        H = rng.choice([2, 4, 8])
        Hkv = H // rng.choice([r for r in (1, 1, 2, 4) if r <= H])
        G = _even(_log_uniform(rng, 48, 1100), rng.choice([0, 0, 64]))
        B, groups = rng.choice([1, 1, 2]), rng.choice([1, 2, 4, 4, 5])
    else:
        D = rng.choice([128, 128, 128, 64])
        H = rng.choice([4, 8, 16, 32, 32, 40, 64])
        Hkv = H // rng.choice([r for r in (1, 1, 1, 2, 4, 8, H) if H % r == 0])
        G = _even(_log_uniform(rng, 128, 25600), rng.choice([0, 0, 128, 256]))
        B, groups = rng.choice([1, 1, 2, 4]), rng.choice([2, 4, 4, 4, 8])
    N = G * groups
    passes = rng.choice(["fwd_bwd", "fwd_bwd", "fwd_bwd", "fwd"])
    call = rng.choice(["tensors", "tensors", "tensors", "full", "variant2", "shard", "static", "shift"])
    shift, heads_total, offset = -1, 0, 0
    if call == "shard":
        heads_total = 4 * H
        offset = (H // Hkv) * rng.randrange(3 * Hkv + 1)
    elif call == "shift":
        shift = rng.randrange(G)
    elif call == "static" and (B * H * N > 1 << 20 or (H // 2) % (H // Hkv)):
        call = "tensors"   # the library's scratch holds the row terms of 2^21 rows and no partial sums
    return _case(None, "f32" if fp32 else "bf16", B, N, H, Hkv, D, G, passes, call, shift, heads_total, offset)


def draw(rng):
    largest = listed()[-1]
    while True:
        c = _draw(rng)
        w, most = work(c), work(largest)
        if c["dtype"] == "f32":
            if c["B"] * c["N"] <= 8192:
                return c
        elif w["flops"] <= most["flops"] and w["bytes"] <= most["bytes"]:
            return c


def prepare(case, seed):
    """q, k, v and the gradient of o as a layer has them: iid N(0, 1), the repository's stand-in
    for activations after rotary embedding.  Outputs, workspace and parameter blocks are
    allocated once and kept, as in a training loop."""
    c = case
    B, N, H, Hkv, D, G = c["B"], c["N"], c["H"], c["Hkv"], c["D"], c["G"]
    dt = DTYPES[c["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(heads):
        return torch.randn((B, N, heads, D), generator=gen, device="cuda", dtype=dt)

    packed = c["call"] == "variant2"
    s = {"case": c, "G": G}
    if packed:
        qkv = normal(H + 2 * Hkv)
        q, k, v = qkv[:, :, :H], qkv[:, :, H:H + Hkv], qkv[:, :, H + Hkv:]
    else:
        q, k, v = normal(H), normal(Hkv), normal(Hkv)
    o = torch.empty((B, N, H, D), device="cuda", dtype=dt)
    lse = torch.empty((B, H, N), device="cuda", dtype=torch.float32)
    s.update(q=q, k=k, v=v, o=o, lse=lse)
    kw = {}
    if c["call"] == "full":
        kw["shift_rule"] = binding.SHIFT_NONE
    elif packed:
        kw.update(wrap_variant=binding.WRAP_SPLIT, strided=True)
    elif c["call"] == "shard":
        kw.update(heads_total=c["heads_total"], head_offset=c["offset"])
    elif c["call"] == "shift":
        kw["shift"] = c["shift"]
    s["fwd"] = binding.make_params(q, k, v, o, lse, G, **kw)
    if c["passes"] == "fwd":
        return s
    s["do"] = do = normal(H)
    if packed:
        s["dqkv"] = dqkv = torch.empty_like(qkv)
        dq, dk, dv = dqkv[:, :, :H], dqkv[:, :, H:H + Hkv], dqkv[:, :, H + Hkv:]
    else:
        dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    ws = None
    if c["call"] != "static":
        p = binding.make_params(q, k, v, o, lse, G, dout=do, dq=dq, dk=dk, dv=dv, **kw)
        ws = torch.empty(binding.bwd_workspace_bytes_ex(p), dtype=torch.uint8, device="cuda")
    s.update(dq=dq, dk=dk, dv=dv, ws=ws)
    s["bwd"] = binding.make_params(q, k, v, o, lse, G, dout=do, dq=dq, dk=dk, dv=dv, workspace=ws, **kw)
    return s


def run(s):
    c = s["case"]
    backward = c["passes"] == "fwd_bwd"
    if c["call"] == "tensors":
        binding.s2attn_fwd(s["q"], s["k"], s["v"], s["o"], s["lse"], s["G"])
        if backward:
            binding.s2attn_bwd(s["q"], s["k"], s["v"], s["o"], s["do"], s["lse"], s["dq"], s["dk"], s["dv"],
                               s["ws"], s["G"])
    else:
        binding.s2attn_fwd_ex(s["fwd"])
        if backward:
            (binding.s2attn_bwd_ex_static if c["call"] == "static" else binding.s2attn_bwd_ex)(s["bwd"])
    out = {"o": s["o"], "lse": s["lse"]}
    if backward:
        out.update({"dqkv": s["dqkv"]} if c["call"] == "variant2" else {"dq": s["dq"], "dk": s["dk"], "dv": s["dv"]})
    return out


def tolerance(case):
    # Against the oracle in 64 bits, worst output over eight shapes of these ranges: fp32 relative
    # error 7.9e-7, largest 8.9e-6; bf16 2.5e-3 (P and dS are rounded to bf16 before the second
    # products, o and the gradients on output), largest 0.15 (single elements of dk).
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 1e-2, "max": 0.5}
