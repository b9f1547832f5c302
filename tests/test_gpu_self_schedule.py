"""Launches in which each item has a workgroup that finds it by itself, against the same sequences in a batch that goes
through the item list: O, LSE and dQ agree bit for bit; and the lists that are built beside such a launch."""
import numpy as np
import pytest
import torch

from oracle import sched_oracle as so
from paper_2412_07894_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

# by the number of heads: as many sequences as leave each item a workgroup
CASES = [[1], [0, 5, 0, 0, 300, 0], [64, 63, 65, 1, 255, 256, 257], [1] * 120, [1023]]
MANY = {1: [[0] * 200 + [129] + [0] * 53 + [17], [2] * 100 + [0] * 155], 2: [[0] * 72 + [129] + [0] * 52 + [17], [2] * 100 + [0] * 26]}
FORMS = [("bf16", 2, 1, 128, None), ("bf16", 1, 1, 64, None), ("bf16", 1, 1, 128, 1e4), ("bf16", 2, 1, 64, 500.0), ("fp32", 2, 2, 64, None), ("fp32", 1, 1, 128, None)]


def preludes(fn):
    """What fn returns, and how many launches were preceded by one that builds their lists."""
    binding.enable_kernel_timing(True)
    try:
        r = fn()
        return r, sum(n == "schedule_prelude" for n, _ in binding.kernel_times())
    finally:
        binding.enable_kernel_timing(False)


@pytest.mark.parametrize("dtype,hq,hkv,d,rope_base,lens", [(*f, x) for f in FORMS for x in CASES + MANY[f[1]]])
def test_own_items_equal_listed_ones(dtype, hq, hkv, d, rope_base, lens):
    dt, code = (torch.bfloat16, binding.HYD_BF16) if dtype == "bf16" else (torch.float32, binding.HYD_FP32)
    T = sum(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(59)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(dt)
    x = (mk(hq), mk(hkv), mk(hkv), mk(hq))
    ws = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, code, 0), dtype=torch.uint8, device="cuda")

    def run(copies, workspace=None):
        n = lens * copies
        cu = torch.from_numpy(wl.cu_seqlens(n)).cuda()
        q, k, v, do = (t.repeat(copies, 1, 1) for t in x)
        o, lse = binding.varlen_attn_fwd(q, k, v, cu, max(n), d ** -0.5, workspace=workspace, rope_base=rope_base)
        dq = binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, max(n), d ** -0.5, rope_base=rope_base)[0]
        return o[:T], lse[:, :T], dq[:T]

    print(f"\n{len(lens)} sequences, {T} tokens, {dtype} {hq}/{hkv} d={d} rope={rope_base}", flush=True)
    small, listed = preludes(lambda: run(1, ws))
    # (a backward in fp32 takes sequences of up to eight tokens from a list)
    assert listed == (dtype == "fp32" and max(lens) <= 8), "the sizes are meant to find their items by themselves"
    tile, rec = binding.schedule_items(ws, T, len(lens), hq, hkv, d, code, 0, 0)
    assert sorted(map(tuple, rec.tolist())) == sorted(so.records(lens, tile))
    assert binding.schedule_status(ws, T, len(lens), hq, hkv, d, code, 0) == 0
    large, listed = preludes(lambda: run(max(257 // len(lens) + 1, 257 // hq + 1)))
    assert listed == (1 if dtype == "bf16" else 2)       # (the bf16 backward's lists come from its preparation)
    for name, a, b in zip(("o", "lse", "dq"), small, large):
        assert bool(torch.isfinite(a.float()).all()) and torch.equal(a, b), name


# more items than compute units: half tiles of equal sequences, the same of more sequences than a wave has lanes, 64-row tiles
@pytest.mark.parametrize("lens,hq", [([2000] * 19, 1), ([200, 0, 130] * 34, 2), ([1100] * 6 + [5], 3)])
def test_own_items_of_a_second_round(lens, hq):
    """They agree bit for bit with listed ones, and the workgroups take the longest first: those of the highest level last
    about as long as each other (sequence by sequence they would be spread over all workgroups)."""
    d, T = 128, sum(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(61)
    q, k, v = (torch.randn((T, hq, d), device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    rec = torch.zeros((3 * 512, 4), dtype=torch.int64, device="cuda")

    def run(copies):
        n = lens * copies
        return binding.varlen_attn_fwd(*(t.repeat(copies, 1, 1) for t in (q, k, v)), torch.from_numpy(wl.cu_seqlens(n)).cuda(), max(n), d ** -0.5)

    print(f"\n{len(lens)} sequences, {T} tokens, {hq} heads", flush=True)
    run(1)
    binding.enable_kernel_timing(True)
    binding.set_wg_trace(rec)
    try:
        o, lse = run(1)
        names = [n for n, _ in binding.kernel_times()]
    finally:
        binding.set_wg_trace(None)
        binding.enable_kernel_timing(False)
    assert names == ["fwd_bf16"]
    r = rec[:512].cpu().numpy()
    took = (r[:, 2] - r[:, 1])[r[:, 3] > 0]
    assert 256 < len(took) <= 448
    first = lens.count(max(lens)) * hq
    assert took[:first].min() > 0.5 * took.max() and took[-len(took) // 4:].mean() < took[:first].mean()
    o2, lse2 = run(257 // len(lens) + 1)
    assert torch.equal(o, o2[:T]) and torch.equal(lse, lse2[:, :T])


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("cu,longest,status,written", [([0, 40, 20, 64], 40, 6, 64), ([0, 30, 60, 60], 40, 6, 60), ([0, 64, 64, 64], 32, 0, 64),
                                                       ([0, 700, 700, 700], 256, 2, 256), ([0, 0, 0, 513], 512, 2, 512)])
def test_malformed_lengths_stay_inside(cu, longest, status, written, dtype, d):
    """A cu_seqlens that decreases, ends early or holds a sequence longer than max_seqlen: every workgroup ends, rows past the bound
    get no item, nothing behind the tensors is written, and the status call says what was wrong: HYD_ERR_SEQLENS, or
    HYD_ERR_SHAPE where the length needs more tiles than the bound (a tile that the bound has is taken whole)."""
    hq, T = 2, max(cu[-1], 64)
    dt, code = (torch.bfloat16, binding.HYD_BF16) if dtype == "bf16" else (torch.float32, binding.HYD_FP32)
    q, k, v = (torch.randn((T, hq, d), device="cuda").to(dt) for _ in range(3))
    room = torch.full((T + 64, hq, d), 3.0, dtype=dt, device="cuda")
    o, lse = room[:T], torch.full((hq, T), 77.0, device="cuda")
    ws = torch.empty(binding.workspace_bytes(T, 3, hq, hq, d, code, 0), dtype=torch.uint8, device="cuda")
    c = torch.tensor(cu, dtype=torch.int32, device="cuda")
    _, listed = preludes(lambda: binding.varlen_attn_fwd(q, k, v, c, longest, d ** -0.5, workspace=ws, out=o, lse=lse))
    assert listed == 0
    got = binding.schedule_status(ws, T, 3, hq, hq, d, code, 0)
    print(cu, dtype, d, binding.status_string(got), flush=True)
    assert got == status
    assert bool((room[written:] == 3.0).all()) and bool((lse[:, written:] == 77.0).all())
    if status != 6:
        assert bool((o[:written] != 3.0).any(-1).all()) and bool((lse[:, :written] != 77.0).all())
