"""The backward of a small batch, whose dK/dV and dQ run in one launch with dO converted to fp16 in LDS, against
the same sequences in a batch large enough for the launches one after the other.  Both convert with the
same power of two, so whole items agree bit for bit; items in parts are sums in another order, whose difference stays
below the rounding of the two results to bf16 (2^-9 of each)."""
import pytest
import torch

from paper_2412_07894_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

BOTH_ROWS = 40960         # (token, head) pairs up to which a batch counts as small


def grads(copies, lens, q, k, v, do, d):
    n = lens * copies
    cu = torch.from_numpy(wl.cu_seqlens(n)).cuda()
    x = [t.repeat(copies, 1, 1) for t in (q, k, v, do)]
    o, lse = binding.varlen_attn_fwd(*x[:3], cu, max(n), d ** -0.5)
    T = sum(lens)
    binding.enable_kernel_timing(True)
    try:
        out = [g[:T].float() for g in binding.varlen_attn_bwd(*x[:3], o, lse, x[3], cu, max(n), d ** -0.5)]
        names = [n for n, _ in binding.kernel_times()]
    finally:
        binding.enable_kernel_timing(False)
    assert ("bwd_both_bf16" in names) == (copies == 1)
    return out, "bwd_sum_parts" not in names          # gradients; whether all items were whole


@pytest.mark.parametrize("lens", [[1], [127, 1, 129, 64], [256, 255, 257, 31, 33], [1025, 640], [2048]])
@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (8, 1, 64), (8, 2, 128), (5, 5, 64)])
@pytest.mark.parametrize("rows", ["even", "uneven"])
def test_small_batches_equal_large_ones(lens, hq, hkv, d, rows):
    T = sum(lens)
    assert T * hq <= BOTH_ROWS
    g = torch.Generator(device="cuda")
    g.manual_seed(43)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)
    if rows == "uneven":          # rows of other sizes, of zeros, below the normal numbers
        f = 2.0 ** -torch.randint(0, 30, (T, hq, 1), device="cuda", generator=g).float()
        f[::7] = 0.0
        f[3::11] = 2.0 ** -130
        f[-1] = 1.0
        do = (do.float() * f).to(torch.bfloat16)
    print(f"\nlens={lens} {hq}/{hkv} d={d} {rows}", flush=True)
    small, whole = grads(1, lens, q, k, v, do, d)
    large, whole2 = grads(BOTH_ROWS // (T * hq) + 1, lens, q, k, v, do, d)
    assert torch.equal(small[0], large[0])
    for name, x, y in zip(("dk", "dv"), small[1:], large[1:]):
        assert bool(torch.isfinite(x).all()) and float((x - y).norm()) <= 2.0 ** -8 * float(y.norm()), name
        assert torch.equal(x, y) or not (whole and whole2), name
    if hq == hkv and T < 400:
        assert whole and whole2, "some of the sizes are meant to be compared bit for bit"


@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 1e9])
def test_a_row_out_of_range_spoils_what_it_reaches(bad):
    """One row of dO that fp16 cannot hold beside ordinary ones: the keys behind it and the other sequences and
    heads are what they are in a large batch."""
    lens, hq, hkv, d = [300, 200], 2, 2, 128
    T = sum(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(47)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)
    do[100, 1, 5] = bad
    small, whole = grads(1, lens, q, k, v, do, d)
    large, whole2 = grads(BOTH_ROWS // (T * hq) + 1, lens, q, k, v, do, d)
    for name, x, y in zip(("dq", "dk", "dv"), small, large):
        ok = torch.isfinite(x)
        assert torch.equal(ok, torch.isfinite(y)), name
        assert float((x[ok] - y[ok]).norm()) <= 2.0 ** -8 * float(y[ok].norm()), name
        assert bool(ok[300:].all()) and bool(ok[:, 0].all()), name


@pytest.mark.parametrize("lens,hq,hkv,d,joint", [([40960], 1, 1, 64, True), ([20480], 2, 1, 128, True), ([10240], 4, 4, 64, True), ([13600], 3, 1, 64, False), ([11000], 3, 1, 64, True),
                                                 ([6800], 6, 2, 128, False), ([1280], 32, 1, 128, False), ([600], 64, 1, 64, False), ([4000], 8, 1, 64, True),
                                                 ([640] * 8, 8, 2, 64, True), ([40961], 1, 1, 64, False)])
def test_which_batches_count_as_small(lens, hq, hkv, d, joint):
    """Up to 40960 (token, head) pairs; with three or more query heads per KV head less for one sequence.  The gradients
    against those of the range variant, which has launches of its own (parts of other lengths: see above)."""
    T, nseq, ml = sum(lens), len(lens), max(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(67)
    q, k, v, do = (torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16) for h in (hq, hkv, hkv, hq))
    cu = torch.from_numpy(wl.cu_seqlens(lens)).cuda()
    o, lse = binding.varlen_attn_fwd(q, k, v, cu, ml, d ** -0.5)
    binding.enable_kernel_timing(True)
    try:
        got = binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, ml, d ** -0.5)
        names = [n for n, _ in binding.kernel_times()]
    finally:
        binding.enable_kernel_timing(False)
    print(f"\n{lens} {hq}/{hkv} d={d}: {names}", flush=True)
    assert ("bwd_both_bf16" in names) == joint
    other = [torch.zeros_like(x) for x in (q, k, v)]
    binding.varlen_attn_bwd_range(q, k, v, o, lse, do, cu, [(0, 1 << 20, 0, 1 << 20)] * nseq, ml, d ** -0.5, *other)
    for name, x, y in zip(("dq", "dk", "dv"), got, other):
        assert float((x.float() - y.float()).norm()) <= 2.0 ** -8 * float(y.float().norm()), name
