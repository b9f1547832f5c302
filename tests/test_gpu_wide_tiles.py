"""dK/dV by tiles of 256 keys, 64 to a wave, against the tiles of 128 that the range variant keeps: over the whole
range both take the same products in the same order, so dK and dV agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2412_07894_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 95, 97, 127, 129, 191, 193, 255, 256, 257, 319, 321, 448, 511, 512, 513, 700, 1025]


@pytest.mark.parametrize("hq,hkv,d,longest,n,scale", [(8, 8, 128, 4095, 12, 1.0), (8, 8, 64, 3000, 8, -1.0), (32, 8, 128, 2049, 16, 1.0), (20, 10, 64, 2111, 8, 1.0),
                                                      (10, 10, 128, 2943, 14, 0.0)])
@pytest.mark.parametrize("special", [False, True])
def test_wide_tiles_equal_narrow_ones(hq, hkv, d, longest, n, scale, special):
    lens = EDGES + [longest] * n
    T, ml = sum(lens), max(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(53)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    if special:             # rows of infinities and NaN: they spoil the keys up to their own block of 32 and no others
        at = np.concatenate([[0], np.cumsum(lens)])
        for s, row, x in ((len(lens) - 1, 640 + 5, float("inf")), (len(lens) - 3, 288, float("nan")), (15, 40, float("inf"))):
            do[int(at[s]) + row, 0] = x
    s = scale * d ** -0.5
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, ml, s)
    ws = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 1), dtype=torch.uint8, device="cuda")
    _, dk, dv = binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, ml, s, workspace=ws)
    tile, _ = binding.executed_items(ws, T, len(lens), hq, hkv, d, binding.HYD_BF16, 1, 0)[:2]
    print(f"\n{hq}/{hkv} d={d} longest={longest} special={special}: tile {tile}", flush=True)
    assert tile == 256, "the sizes are meant to take the wide form"
    full = [(0, 1 << 20, 0, 1 << 20)] * len(lens)
    narrow = [torch.zeros_like(x) for x in (q, k, v)]
    binding.varlen_attn_bwd_range(q, k, v, o, lse, do, cu, full, ml, s, *narrow)
    for name, x, y in zip(("dk", "dv"), (dk, dv), narrow[1:]):
        ok = torch.isfinite(y.float())
        assert torch.equal(ok, torch.isfinite(x.float())) and torch.equal(x[ok], y[ok]), name
        assert bool(ok.all()) != special
        assert bool((x[ok] != 0).any()) or scale == 0.0


@pytest.mark.parametrize("lens,hq,hkv,d,tile", [([700] * 17 + [100], 32, 8, 128, 128), ([1000] * 24, 32, 8, 128, 256), ([640] * 25 + [384], 32, 8, 128, 128), ([500] * 24, 16, 8, 64, 128),
                                                ([1500] * 8, 16, 8, 64, 256), ([500] * 100, 32, 32, 64, 256), ([1500] * 8, 40, 40, 128, 256), ([2500] * 5, 10, 10, 128, 128),
                                                ([3713], 32, 32, 128, 128), ([7000], 32, 32, 128, 256), ([2743], 48, 48, 64, 128), ([4700], 48, 48, 64, 256)])
def test_wide_where_items_are_long_and_many(lens, hq, hkv, d, tile):
    """dK and dV against the range variant, which keeps the narrow form: the same products in the same order."""
    T, ml = sum(lens), max(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(59)
    q, k, v, do = (torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16) for h in (hq, hkv, hkv, hq))
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, ml, d ** -0.5)
    ws = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 1), dtype=torch.uint8, device="cuda")
    _, dk, dv = binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, ml, d ** -0.5, workspace=ws)
    got = binding.executed_items(ws, T, len(lens), hq, hkv, d, binding.HYD_BF16, 1, 0)[0]
    print(f"\n{len(lens)} x {ml} {hq}/{hkv} d={d}: tile {got}", flush=True)
    assert got == tile
    other = [torch.zeros_like(x) for x in (q, k, v)]
    binding.varlen_attn_bwd_range(q, k, v, o, lse, do, cu, [(0, 1 << 20, 0, 1 << 20)] * len(lens), ml, d ** -0.5, *other)
    assert torch.equal(dk, other[1]) and torch.equal(dv, other[2])


# (bound, form): equal lengths that need no look at them; short ones under a bound; a few long ones among short ones; one long and all others alike, that the bound hides
@pytest.mark.parametrize("lens,hq,hkv,d,bound,tile", [([1500] * 16, 32, 8, 128, 1500, 256), ([128] * 256, 32, 32, 128, 8192, 128), ([500] * 66, 8, 8, 64, 33000, 128), ([300] * 100, 32, 8, 128, 30000, 128),
                                                      ([128] * 200 + [9000, 7000, 5000, 4000], 32, 32, 128, 9000, 256), ([128] * 200 + [9000, 7000, 5000, 4000], 32, 32, 128, 50600, 256),
                                                      ([64] * 100 + [11000], 8, 8, 128, 17400, 128), ([0] * 30 + [40] * 5 + [3000] * 9 + [0], 16, 16, 64, 27200, 256)])
@pytest.mark.parametrize("host", [False, True])
def test_bound_above_the_lengths(lens, hq, hkv, d, bound, tile, host):
    """max_seqlen may be any bound: where it would decide, the lengths on the device do (or a host copy of them), and of the
    two lists one is left empty; dK and dV are those of the range variant, several times with one workspace."""
    T, nseq = sum(lens), len(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(73)
    q, k, v, do = (torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16) for h in (hq, hkv, hkv, hq))
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    at = [int(x) for x in wl.cu_seqlens(lens)] if host else None
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, bound, d ** -0.5)
    ws = torch.full((binding.workspace_bytes(T, nseq, hq, hkv, d, binding.HYD_BF16, 1),), 0xff, dtype=torch.uint8, device="cuda")
    other = [torch.zeros_like(x) for x in (q, k, v)]
    binding.varlen_attn_bwd_range(q, k, v, o, lse, do, cu, [(0, 1 << 20, 0, 1 << 20)] * nseq, max(lens), d ** -0.5, *other)
    for _ in range(2):
        grads = [torch.full_like(x, float("nan")) for x in (q, k, v)]
        binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, bound, d ** -0.5, cu_seqlens_host=at, workspace=ws, dq=grads[0], dk=grads[1], dv=grads[2])
        got, _, rec = binding.executed_items(ws, T, nseq, hq, hkv, d, binding.HYD_BF16, 1, 0)
        print(f"\n{nseq} sequences, longest {max(lens)}, bound {bound}, {hq}/{hkv} d={d}: tile {got}, {len(rec)} items", flush=True)
        assert got == tile and len(rec) == sum(-(-n // tile) for n in lens)
        assert torch.equal(grads[1], other[1]) and torch.equal(grads[2], other[2])


@pytest.mark.parametrize("hq,hkv,d", [(40, 40, 128), (32, 8, 128), (32, 8, 64)])
def test_rotary_positions(hq, hkv, d):
    """Sequences that take the wide form, and the same beside many short ones, where the narrow form is taken: bit for bit."""
    long = [1500, 1499, 1473, 1535] * 2
    g = torch.Generator(device="cuda")
    g.manual_seed(79)
    x = [torch.randn((40000, h, d), device="cuda", generator=g).to(torch.bfloat16) for h in (hq, hkv, hkv, hq)]
    got = []
    for lens, tile in ((long, 256), (long + [64] * 380, 128)):
        T, ml = sum(lens), max(lens)
        q, k, v, do = (t[:T] for t in x)
        cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
        o, lse = binding.varlen_attn_fwd(q, k, v, cu, ml, d ** -0.5, rope_base=1e4)
        ws = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 1), dtype=torch.uint8, device="cuda")
        got.append([r[:sum(long)] for r in binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, ml, d ** -0.5, workspace=ws, rope_base=1e4)])
        taken = binding.executed_items(ws, T, len(lens), hq, hkv, d, binding.HYD_BF16, 1, 0)[0]
        print(f"\n{hq}/{hkv} d={d} {len(lens)} sequences: tile {taken}", flush=True)
        assert taken == tile
    for name, a, b in zip(("dq", "dk", "dv"), *got):
        assert bool(torch.isfinite(a.float()).all()) and torch.equal(a, b), name
