"""Performance cases of the packed variable-length causal attention library.

A case is one call pattern of a training or prefill program over one packed buffer:

    call     "fwd"   forward alone (prefill, evaluation)
             "bwd"   backward alone, O and LSE from an earlier forward
             "step"  forward, then backward: the unit the latency model of the planner prices
             "rope"  K rotated by its own pass, forward and backward with Q rotated inside the
                     kernels, dK turned back: a layer with rotary positions reset per sequence
             "ring"  what one rank of a context-parallel group does for its query chunk: a forward
                     visit per key chunk merged into the running result, then a backward visit
                     per key chunk
    dtype    "bf16" (training) or "fp32" (numerical checks of a model)
    lens     how the buffer is filled (see `lengths`), `tokens` its size
    hq, hkv, d   head counts and head dimension (hq / hkv > 1: grouped-query attention)

Everything a program would keep from call to call (workspaces, outputs, cu_seqlens on the device)
is made in `prepare`, as bench.py does.
"""
import math
import random

import torch

from paper_2412_07894_amd import binding
from paper_2412_07894_amd import workloads as wl

ROPE_BASE = 10000.0


def _case(name, call, dtype, lens, tokens, hq, hkv, d, seed=0, cp=0, rank=0):
    c = {"call": call, "dtype": dtype, "lens": lens, "tokens": tokens, "hq": hq, "hkv": hkv, "d": d, "seed": seed,
         "cp": cp, "rank": rank}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: one short prompt pack, and the tiny fp32 batch of a numerical check
        _case("fwd_prompts_256", "fwd", "bf16", "config1", 256, 32, 8, 128),
        _case("step_fp32_tiny", "step", "fp32", "config1", 256, 2, 2, 64),
        # a small micro-batch on one rank of a tensor-parallel group (32 heads over 4 ranks)
        _case("step_tp_shard_2k", "step", "bf16", "lognormal", 2048, 8, 8, 128, seed=3),
        # fp32 at the size of a real sequence mix: gradient checks against the bf16 path
        _case("step_fp32_4k", "step", "fp32", "lognormal", 4001, 8, 8, 128, seed=5),
        # a buffer of nothing but short sequences (what most packed buffers of a corpus hold)
        _case("step_short_32k", "step", "bf16", "short", 32768, 32, 8, 128, seed=1),
        # one micro-batch of log-normal lengths, multi-head attention: the ordinary training step
        _case("step_lognormal_16k", "step", "bf16", "config2", 16384, 32, 32, 128),
        # the same kind of step with rotary positions and grouped heads, ragged buffer size
        _case("rope_lognormal_15k", "rope", "bf16", "lognormal", 15001, 32, 8, 128, seed=4),
        # head_dim 64, heavy-tailed lengths
        _case("step_d64_pareto_32k", "step", "bf16", "pareto", 32768, 32, 32, 64, seed=4),
        # the last rank of a context-parallel ring of four on one long sequence and some short ones
        _case("ring_cp4_16k", "ring", "bf16", "longmix", 16384, 32, 8, 128, seed=6, cp=4, rank=3),
        # forward over four buffers of heavy-tailed lengths, 40 heads
        _case("fwd_pareto_4x32k", "fwd", "bf16", "config3", 131072, 40, 40, 128),
        # backward over eight buffers, one 32768-token sequence among 409 short ones
        _case("bwd_imbalance_8x32k", "bwd", "bf16", "config4", 262144, 32, 8, 128),
        # long contexts, 64 query heads on 8 KV heads: the largest step
        _case("step_longctx_2x64k", "step", "bf16", "config5", 131072, 64, 8, 128),
    ]


_HEADS = [(32, 32), (40, 40), (32, 8), (64, 8), (8, 8), (8, 1), (10, 10), (16, 2), (5, 5)]
_LENS = ["equal", "lognormal", "pareto", "short", "imbalance", "longmix", "single"]


def draw(rng):
    call = rng.choice(["fwd", "bwd", "step", "step", "step", "rope", "ring"])
    dtype = "fp32" if call in ("fwd", "bwd", "step") and rng.random() < 0.15 else "bf16"
    lens = rng.choice(_LENS)
    if call == "ring":
        lens = rng.choice(["longmix", "single", "imbalance"])
    lo, hi = (64, 4096) if dtype == "fp32" else ((2048, 65536) if call == "ring" else (64, 131072))
    tokens = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        tokens |= 1
    if dtype == "fp32":
        hq, hkv = rng.choice([(2, 2), (4, 2), (8, 8), (8, 2)])
    else:
        hq, hkv = rng.choice(_HEADS)
    d = rng.choice([64, 128]) if dtype == "fp32" else rng.choice([128, 128, 128, 64])
    cp = rng.choice([2, 4]) if call == "ring" else 0
    rank = rng.randrange(1, cp) if cp else 0
    seed = rng.randrange(1 << 20)
    # no dearer than the largest listed case of its dtype
    top = {"bf16": 14.0 * 128 * 64 * 6.3e8, "fp32": 14.0 * 128 * 8 * wl.causal_pairs(lengths(listed()[3]))}[dtype]
    while True:
        case = _case(None, call, dtype, lens, tokens, hq, hkv, d, seed, cp, rank)
        if work(case)["flops"] <= top:
            return case
        tokens = tokens * 2 // 3


def lengths(case):
    """Sequence lengths of the case's packed buffer; they sum to `tokens`."""
    kind, T = case["lens"], case["tokens"]
    if kind.startswith("config"):
        return [int(x) for x in wl.seqlens(int(kind[6:]))]
    rng = random.Random(case["seed"])
    if kind == "single":
        return [T]
    if kind == "equal":                          # copies of one (mostly odd) length, the rest ragged
        one = int(round(math.exp(rng.uniform(math.log(16), math.log(4096)))))

        def nxt():
            return one
    elif kind == "lognormal":                    # as configuration 2: median 1024
        def nxt():
            return max(32, int(round(math.exp(rng.gauss(math.log(1024.0), 1.0)))))
    elif kind == "pareto":                       # as configuration 3
        def nxt():
            return min(32768, int(128.0 * (1.0 - rng.random()) ** (-1.0 / 1.2)))
    elif kind == "short":                        # as configuration 4's short buffers
        def nxt():
            return rng.randint(64, 1024)
    elif kind == "imbalance":                    # one sequence of half the buffer, then short ones
        first = [max(1, T // 2)]

        def nxt():
            return first.pop() if first else rng.randint(64, 1024)
    elif kind == "longmix":                      # as configuration 5, in proportion to the buffer
        def nxt():
            u = rng.random()
            a, b = (32, T // 16) if u < 0.6 else ((T // 16, T // 4) if u < 0.9 else (T // 4, T))
            return max(1, rng.randint(min(a, b), max(a, b)))
    else:
        raise ValueError(kind)
    out, room = [], T
    while room > 0:
        n = min(nxt(), room)
        out.append(n)
        room -= n
    return out


def _chunks(L, cp):
    """Bounds of the cp chunks of a sequence: multiples of the range granule, the last one open."""
    g = binding.RANGE_ALIGN
    per = max(-(-(-(-L // cp)) // g) * g, g)
    return [(c * per, (c + 1) * per if c + 1 < cp else max(L, cp * per)) for c in range(cp)]


def _ranges(lens, cp, rank, c):
    out = []
    for L in lens:
        b = _chunks(L, cp)
        out.append((b[rank][0], b[rank][1], b[c][0], b[c][1]))
    return out


def prepare(case, seed):
    lens = lengths(case)
    T, hq, hkv, d = case["tokens"], case["hq"], case["hkv"], case["d"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    code = binding.HYD_BF16 if case["dtype"] == "bf16" else binding.HYD_FP32
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def rnd(h):                                  # i.i.d. N(0, 1), the input recipe of every configuration
        return torch.randn((T, h, d), device="cuda", dtype=torch.float32, generator=g).to(dt)

    st = {"call": case["call"], "scale": 1.0 / math.sqrt(d), "max_len": max(lens)}
    st["q"], st["k"], st["v"] = rnd(hq), rnd(hkv), rnd(hkv)
    st["cu"] = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    st["ws_f"] = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, code, 0), dtype=torch.uint8, device="cuda")
    ring = case["call"] == "ring"
    make = torch.zeros_like if ring else torch.empty_like          # a ring visit leaves other ranks' rows alone
    st["o"] = make(st["q"])
    st["lse"] = torch.zeros((hq, T), dtype=torch.float32, device="cuda")
    if case["call"] != "fwd":
        st["do"] = rnd(hq)
        st["ws_b"] = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, code, 1), dtype=torch.uint8, device="cuda")
        st["dq"], st["dk"], st["dv"] = make(st["q"]), make(st["k"]), make(st["v"])
    if case["call"] == "bwd":
        binding.varlen_attn_fwd(st["q"], st["k"], st["v"], st["cu"], st["max_len"], st["scale"], workspace=st["ws_f"],
                                out=st["o"], lse=st["lse"])
    if case["call"] == "rope":
        st["k_rot"], st["dk_rot"] = torch.empty_like(st["k"]), torch.empty_like(st["k"])
    if ring:
        cp, rank = case["cp"], case["rank"]
        st["visits"] = [_ranges(lens, cp, rank, c) for c in range(rank, -1, -1)]      # own chunk first, then the arriving ones
        st["part_o"], st["part_lse"] = torch.zeros_like(st["o"]), torch.full_like(st["lse"], float("-inf"))
        st["grads"] = [(st["dq"], st["dk"], st["dv"])] + [(make(st["q"]), make(st["k"]), make(st["v"])) for _ in range(rank)]
    return st


def run(st):
    call, q, k, v, cu, ml, scale = st["call"], st["q"], st["k"], st["v"], st["cu"], st["max_len"], st["scale"]
    o, lse = st["o"], st["lse"]
    if call == "fwd":
        return binding.varlen_attn_fwd(q, k, v, cu, ml, scale, workspace=st["ws_f"], out=o, lse=lse)
    do, dq, dk, dv = st["do"], st["dq"], st["dk"], st["dv"]
    if call == "bwd":
        return binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, ml, scale, workspace=st["ws_b"], dq=dq, dk=dk, dv=dv)
    if call == "step":
        binding.varlen_attn_fwd(q, k, v, cu, ml, scale, workspace=st["ws_f"], out=o, lse=lse)
        binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, ml, scale, workspace=st["ws_b"], dq=dq, dk=dk, dv=dv)
        return o, lse, dq, dk, dv
    if call == "rope":
        kr, dkr = st["k_rot"], st["dk_rot"]
        binding.rope_packed(k, cu, ROPE_BASE, out=kr)
        binding.varlen_attn_fwd(q, kr, v, cu, ml, scale, workspace=st["ws_f"], out=o, lse=lse, rope_base=ROPE_BASE)
        binding.varlen_attn_bwd(q, kr, v, o, lse, do, cu, ml, scale, workspace=st["ws_b"], dq=dq, dk=dkr, dv=dv, rope_base=ROPE_BASE)
        binding.rope_packed(dkr, cu, ROPE_BASE, inverse=True, out=dk)
        return o, lse, dq, dk, dv
    # ring: the rank's own chunk writes the running result, every other visit is merged into it
    po, pl = st["part_o"], st["part_lse"]
    for i, ranges in enumerate(st["visits"]):
        if i == 0:
            binding.varlen_attn_fwd_range(q, k, v, cu, ranges, ml, scale, o, lse, workspace=st["ws_f"])
        else:
            binding.varlen_attn_fwd_range(q, k, v, cu, ranges, ml, scale, po, pl, workspace=st["ws_f"])
            binding.attn_merge(o, lse, po, pl, out=o, lse_out=lse)
    for ranges, (gq, gk, gv) in zip(st["visits"], st["grads"]):
        binding.varlen_attn_bwd_range(q, k, v, o, lse, do, cu, ranges, ml, scale, gq, gk, gv, workspace=st["ws_b"])
    return o, lse, st["grads"]


def _visible(L, cp, rank, c):
    """(query, key) pairs of query chunk `rank` and key chunk c <= rank of a sequence, its query rows, its key rows."""
    b = _chunks(L, cp)
    nq = max(0, min(b[rank][1], L) - b[rank][0])
    nk = max(0, min(b[c][1], L) - b[c][0])
    return (nq * (nq + 1) // 2 if c == rank else nq * nk), nq, nk


def work(case):
    lens = lengths(case)
    T, hq, hkv, d, call = case["tokens"], case["hq"], case["hkv"], case["d"], case["call"]
    el = 2 if case["dtype"] == "bf16" else 4
    row_q, row_kv = hq * d * el, hkv * d * el
    if call == "ring":
        flops = bytes_ = 0.0
        for c in range(case["rank"] + 1):
            for L in lens:
                pairs, nq, nk = _visible(L, case["cp"], case["rank"], c)
                if pairs:
                    flops += 14.0 * d * hq * pairs
                    # forward: q, k, v in, o and lse out; backward: q, o, dO, lse, k, v in, dq, dk, dv out
                    bytes_ += nq * (2 * row_q + 4 * hq) + nk * 2 * row_kv
                    bytes_ += nq * (4 * row_q + 4 * hq) + nk * 4 * row_kv
                if c != case["rank"]:                # merge: two partials of the rank's rows in, one out
                    bytes_ += nq * 3 * (row_q + 4 * hq)
        return {"bytes": bytes_, "flops": flops}
    pairs = wl.causal_pairs(lens)
    fwd = (4.0 * d * hq * pairs, T * (2 * row_q + 2 * row_kv + 4 * hq))
    bwd = (10.0 * d * hq * pairs, T * (4 * row_q + 4 * row_kv + 4 * hq))
    parts = {"fwd": [fwd], "bwd": [bwd], "step": [fwd, bwd],
             "rope": [fwd, bwd, (0.0, 4.0 * T * row_kv)]}[call]
    return {"bytes": float(sum(p[1] for p in parts)), "flops": float(sum(p[0] for p in parts))}


def tolerance(case):
    # four times what the path shows against itself in 64 bits (relative 2-norm): bf16 outputs 2.1e-3
    # at most, a ring 3.3e-3 (its partial results are rounded to bf16 at every merge), fp32 7.7e-7
    if case["dtype"] == "fp32":
        return {"rel": 3e-6}
    return {"rel": 1.3e-2 if case["call"] == "ring" else 8e-3}
