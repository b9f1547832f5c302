"""dK/dV items taken in parts (few KV heads or few tokens): fp32 sums of the parts added in a pass of
their own.  Against the fp64 oracle with the bars of the other parity tests, over the number of parts, the
remainders of steps per part, and the range variant; twice the same bits; rows that get no item stay."""
import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc
from paper_2412_07894_amd import binding, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def setup(lens, hq, hkv, d, seed):
    cu, q, k, v, do = wl.custom(lens, hq, hkv, d, "bf16", seed)
    if hq // hkv > 16:          # a sum over 32 heads reaches 12, where rounding to bf16 alone (2^-5 above 8) passes
        do = do * 0.25          # the absolute bar of 2e-2; the gradients follow a power of two exactly
    scale = 1.0 / float(np.sqrt(d))
    dev = [gu.to_dev(x, "bf16") for x in (q, k, v, do)]
    cu_d = torch.from_numpy(cu).cuda()
    o, lse = binding.varlen_attn_fwd(*dev[:3], cu_d, max(lens), scale)
    return cu, (q, k, v, do), scale, dev, cu_d, o, lse


def names_of(run):
    binding.enable_kernel_timing(True)
    try:
        run()
        return [n for n, _ in binding.kernel_times()]
    finally:
        binding.enable_kernel_timing(False)


@pytest.mark.parametrize("lens,hq,hkv,d,parts", [
    ([1300, 7, 129], 8, 1, 128, True), ([1300, 7, 129], 16, 2, 64, True), ([2200], 4, 4, 64, True), ([257, 1000], 32, 8, 128, True),
    ([3, 900, 128], 6, 2, 128, True), ([100, 31], 8, 8, 128, False), ([128, 127], 32, 1, 64, True)])
def test_items_in_parts_match_the_oracle(lens, hq, hkv, d, parts):
    print(f"\nparts: {lens} {hq}/{hkv} d = {d}", flush=True)
    cu, host, scale, (q, k, v, do), cu_d, o, lse = setup(lens, hq, hkv, d, 71)
    run = lambda: binding.varlen_attn_bwd(q, k, v, o, lse, do, cu_d, max(lens), scale)
    assert ("bwd_sum_parts" in names_of(run)) == parts
    (dq, dk, dv), again = run(), run()
    for x, y in zip((dq, dk, dv), again):
        assert torch.equal(x, y)
    rdq, rdk, rdv = orc.bwd(*host, cu, scale)
    for name, got, ref in (("dq", dq, rdq), ("dk", dk, rdk), ("dv", dv, rdv)):
        gu.check(name, gu.to_np(got), ref, "bf16")


def test_items_in_parts_of_a_key_range():
    lens, hq, hkv, d = [1500, 300], 8, 1, 128
    cu, host, scale, (q, k, v, do), cu_d, o, lse = setup(lens, hq, hkv, d, 72)
    _, rdk, rdv = orc.bwd(*host, cu, scale)
    ranges = torch.tensor([[0, 4096, 256, 1024], [0, 4096, 256, 1024]], dtype=torch.int32, device="cuda")
    dq, dk, dv = (torch.full_like(x, 7.0) for x in (q, k, v))
    run = lambda: binding.varlen_attn_bwd_range(q, k, v, o, lse, do, cu_d, ranges, max(lens), scale, dq=dq, dk=dk, dv=dv)
    assert "bwd_sum_parts" in names_of(run)
    inside = np.r_[256:1024, 1756:1800]
    outside = np.setdiff1d(np.arange(1800), inside)
    for name, got, ref in (("dk", dk, rdk), ("dv", dv, rdv)):
        got = gu.to_np(got)
        gu.check(name, got[inside], ref[inside], "bf16")
        assert np.all(got[outside] == 7.0), name


@pytest.mark.parametrize("room", [0, 1, 3, 8])
def test_a_smaller_workspace_takes_fewer_parts(room):
    """A workspace with room for the sums of `room` parts (this batch can use eight): right results whatever the number, no parts without."""
    lens, hq, hkv, d = [1300, 7, 129], 8, 1, 128
    T = sum(lens)
    cu, host, scale, (q, k, v, do), cu_d, o, lse = setup(lens, hq, hkv, d, 73)
    part, full = 8 * T * hkv * d, binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 1)
    ws = torch.empty(full - (8 - room) * part + 65536, dtype=torch.uint8, device="cuda")
    ws[-65536:] = 0x5a
    run = lambda: binding.varlen_attn_bwd(q, k, v, o, lse, do, cu_d, max(lens), scale, workspace=ws[:-65536])
    assert ("bwd_sum_parts" in names_of(run)) == (room > 1)
    _, dk, dv = run()
    _, rdk, rdv = orc.bwd_given(*host, gu.to_np(o).astype(np.float32), gu.to_np(lse).astype(np.float32), cu, scale)     # of the stored O and LSE
    gu.check("dk", gu.to_np(dk), rdk, "bf16")
    gu.check("dv", gu.to_np(dv), rdv, "bf16")
    assert bool((ws[-65536:] == 0x5a).all())


def test_no_sums_are_added_where_no_item_was_cut():
    """A decreasing cu_seqlens that holds the same rows twice asks for 16 items of 128 keys, and there are records for
    12: items stay whole although the host expected parts, and the last two tiles get none.  dK and dV are what dK/dV
    wrote, not sums of whatever the workspace held.  Nothing is written behind the workspace."""
    T, hq, hkv, d, n, done = 1000, 8, 1, 128, 4, 768
    cu = torch.tensor([0, T, 0, T, 0], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(41)
    mk = lambda h: torch.randn((T, h, d), device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, do = mk(hq), mk(hkv), mk(hkv), mk(hq)
    one = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    o, lse = binding.varlen_attn_fwd(q, k, v, one, T, d ** -0.5)
    _, rdk, rdv = binding.varlen_attn_bwd(q, k, v, o, lse, do, one, T, d ** -0.5)
    size = binding.workspace_bytes(T, n, hq, hkv, d, binding.HYD_BF16, 1)
    ws = torch.full((size + 65536,), 0xff, dtype=torch.uint8, device="cuda")      # every float of it is a NaN
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    run = lambda: binding.varlen_attn_bwd(q, k, v, o, lse, do, cu, T, d ** -0.5, workspace=ws[:size], dk=dk, dv=dv)
    assert "bwd_sum_parts" in names_of(run)
    assert binding.schedule_status(ws, T, n, hq, hkv, d, binding.HYD_BF16, 1) == 6
    for x, ref in ((dk, rdk), (dv, rdv)):                  # (rounded once in both cases: 2^-9 of each element)
        assert torch.isfinite(x.float()).all() and bool((x[done:] == 0).all())
        assert float((x[:done].double() - ref[:done].double()).norm() / ref[:done].double().norm()) < 2.0 ** -8
    assert bool((ws[size:] == 0xff).all())
