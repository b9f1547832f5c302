"""Items of the forward and dQ kernels that take four query heads of 64 rows each (query heads in
groups of four or eight) against items of one head and 256 rows: the same query heads with their KV
heads repeated run as ungrouped ones.  Every row does the same arithmetic either way, so O, LSE and
dQ agree bit for bit; dK and dV, which stream what the dQ kernel wrote, are the sum over the group,
here rounded once per head to bf16 (2^-9 of each summand, in the 2-norm below 2^-8 of the sum)."""
import pytest
import torch

from paper_2412_07894_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 127, 129, 191, 193, 255, 256, 257, 320, 321, 700, 1025]


@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (8, 1, 64), (16, 2, 128), (32, 8, 128), (32, 8, 64), (12, 3, 128)])
@pytest.mark.parametrize("call", ["plain", "rope"])
def test_split_heads_equal_repeated_kv_heads(hq, hkv, d, call):
    lens = EDGES * (1 + 131072 // (hq * sum(EDGES)))          # enough (token, head) pairs for split items
    T, ml, G = sum(lens), max(lens), hq // hkv
    print(f"\n{call}: {hq}/{hkv} heads, d = {d}, T = {T}", flush=True)
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(23)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)

    def run(kk, vv):
        o, dq = torch.zeros_like(q), torch.zeros_like(q)
        lse = torch.zeros((hq, T), dtype=torch.float32, device="cuda")
        dk, dv = torch.zeros_like(kk), torch.zeros_like(vv)
        s = d ** -0.5
        if call == "rope":
            binding.varlen_attn_fwd(q, kk, vv, cu, ml, s, out=o, lse=lse, rope_base=1e4)
            binding.varlen_attn_bwd(q, kk, vv, o, lse, do, cu, ml, s, dq=dq, dk=dk, dv=dv, rope_base=1e4)
        else:
            binding.varlen_attn_fwd(q, kk, vv, cu, ml, s, out=o, lse=lse)
            binding.varlen_attn_bwd(q, kk, vv, o, lse, do, cu, ml, s, dq=dq, dk=dk, dv=dv)
        return o, lse, dq, dk, dv

    split = run(k, v)
    whole = run(*(x.repeat_interleave(G, dim=1).contiguous() for x in (k, v)))
    for name, x, y in zip(("o", "lse", "dq"), split, whole):
        assert torch.equal(x, y), name
        assert torch.isfinite(x.float()).all() and bool((x != 0).any()), name
    for name, x, y in zip(("dk", "dv"), split[3:], whole[3:]):
        ref = y.view(T, hkv, G, d).double().sum(2)
        rel = float((x.double() - ref).norm() / ref.norm())
        assert rel < 2.0 ** -8, (name, rel)


@pytest.mark.parametrize("copies", [1, 13])
@pytest.mark.parametrize("max_seqlen", [100, 256, 300, 1000])
def test_a_bound_below_the_longest_sequence_covers_whole_tiles(max_seqlen, copies):
    """A sequence longer than max_seqlen gets its first ceil(max_seqlen / 256) tiles of 256 rows, with
    split heads and half tiles as without."""
    lens, hq, hkv, d = [1000, 40, 256] * copies, 8, 2, 128
    T = sum(lens)
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(29)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v = mk(hq), mk(hkv), mk(hkv)
    full, _ = binding.varlen_attn_fwd(q, k, v, cu, max(lens), d ** -0.5)
    o = torch.full_like(q, 7.0)
    binding.varlen_attn_fwd(q, k, v, cu, max_seqlen, d ** -0.5, out=o)
    covered = min(1000, -(-max_seqlen // 256) * 256)
    assert torch.equal(o[:covered], full[:covered]) and torch.equal(o[1000:1296], full[1000:1296])
    assert bool((o[covered:1000] == 7.0).all())


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (3, 1, 64), (8, 2, 128)])
@pytest.mark.parametrize("rope_base", [None, 1e4])
def test_half_tiles_equal_the_tiles_of_a_larger_batch(hq, hkv, d, rope_base):
    """A batch below the limit of the 128-row items against the same sequences in a batch far above it."""
    T = sum(EDGES)
    copies = 1 + 600000 // (T * hq)
    g = torch.Generator(device="cuda")
    g.manual_seed(31)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)

    def run(n):
        lens = EDGES * n
        cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
        x = [t.repeat(n, 1, 1) for t in (q, k, v, do)]
        o, lse = binding.varlen_attn_fwd(*x[:3], cu, max(lens), d ** -0.5, rope_base=rope_base)
        dq, dk, dv = binding.varlen_attn_bwd(*x[:3], o, lse, x[3], cu, max(lens), d ** -0.5, rope_base=rope_base)
        return o[:T], lse[:, :T], dq[:T], dk[:T], dv[:T]

    small, large = run(1), run(copies)
    for name, x, y in zip(("o", "lse", "dq"), small, large):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y), name
    for name, x, y in zip(("dk", "dv"), small[3:], large[3:]):       # sums in another order, rounded to bf16
        rel = float((x.double() - y.double()).norm() / y.double().norm())
        assert rel < 2.0 ** -8, (name, rel)


def test_lists_with_levels_inside_and_outside_lds():
    """With max_seqlen = T the lists of 64-row and 128-row tiles have more levels than fit LDS and the list of
    whole tiles has not; all of them are right, and the bound does not change a bit."""
    from oracle import sched_oracle as so
    lens, hq, hkv, d = [640, 511, 769] * 370, 4, 1, 64
    T, code = sum(lens), binding.HYD_BF16
    assert 4096 * 128 < T < 4096 * 256
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(37)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g, dtype=torch.float32).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)
    size = binding.workspace_bytes(T, len(lens), hq, hkv, d, code, 1)
    out = []
    for bound in (T, max(lens)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        o, lse = binding.varlen_attn_fwd(q, k, v, cu, bound, d ** -0.5)
        out.append((o, lse) + tuple(binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, bound, d ** -0.5, workspace=ws)))
        for which in (0, 1):
            tile, rec = binding.schedule_items(ws, T, len(lens), hq, hkv, d, code, 1, which)
            assert sorted(map(tuple, rec.tolist())) == sorted(so.records(lens, tile)), (bound, which)
    for x, y in zip(*out):
        assert torch.equal(x, y)
