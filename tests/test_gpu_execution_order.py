"""The cheap end of the item list is handed out sequence by sequence when that pays (many short
sequences, no grouped heads).  The order must be a permutation of the list and must not change a bit:
a batch large enough for it equals, bit for bit, its sequences in batches too small for it."""
import numpy as np
import pytest
import torch

from paper_2412_07894_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


def run(q, k, v, do, lens, scale):
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    full = lambda x: torch.full_like(x, float("nan"))
    o, lse = full(q), torch.full((q.shape[1], q.shape[0]), float("nan"), dtype=torch.float32, device="cuda")
    binding.varlen_attn_fwd(q, k, v, cu, max(lens), scale, out=o, lse=lse)
    dq, dk, dv = binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, max(lens), scale, dq=full(q), dk=full(k), dv=full(v))
    return o, lse.t(), dq, dk, dv


@pytest.mark.parametrize("lo,hi,n,dtype", [(1, 1100, 240, "bf16"), (1024, 1024, 160, "bf16"), (30, 200, 900, "bf16"), (1, 400, 120, "fp32")])
def test_grouped_order_equals_small_batches(lo, hi, n, dtype):
    heads, d = 16, 64
    lens = [int(x) for x in np.random.default_rng(3).integers(lo, hi + 1, size=n)]
    T = sum(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, do = (torch.randn((T, heads, d), device="cuda", generator=g).to(dt) for _ in range(4))
    do = do.clamp(-3.9, 3.9)
    at = np.concatenate([[0], np.cumsum(lens)])
    do[torch.from_numpy(at[:-1]).cuda(), 0, 0] = 4.0     # every batch scales dO by the same power of two
    whole = run(q, k, v, do, lens, d ** -0.5)
    for x in whole:
        assert torch.isfinite(x.float()).all()
    step = 10
    for s in range(0, n, step):
        a, b = int(at[s]), int(at[min(s + step, n)])
        part = run(*(x[a:b].contiguous() for x in (q, k, v, do)), lens[s:s + step], d ** -0.5)
        for name, x, y in zip(("o", "lse", "dq", "dk", "dv"), whole, part):
            assert torch.equal(x[a:b], y), (name, s)


def test_records_stay_in_the_workspace_when_seqlens_decrease():
    """A decreasing cu_seqlens can ask for more items than the workspace has records for.  Nothing may be
    written behind it, and the findings are read back."""
    T, heads, d, n = 1000, 32, 64, 200
    cu = torch.tensor([0] + [T if i % 2 == 0 else 0 for i in range(n)], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(19)
    q, k, v = (torch.randn((T, heads, d), device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    need = binding.workspace_bytes(T, n, heads, heads, d, binding.HYD_BF16, 0)
    ws = torch.full((need + 65536,), 0x5a, dtype=torch.uint8, device="cuda")
    binding.varlen_attn_fwd(q, k, v, cu, T, d ** -0.5, workspace=ws)
    assert binding.schedule_status(ws, T, n, heads, heads, d, binding.HYD_BF16, 0) == 6
    assert bool((ws[need:] == 0x5a).all())
