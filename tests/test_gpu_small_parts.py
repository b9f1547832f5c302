"""dK/dV items of a small batch in parts beside dQ: as fine as the batch asks for, and as the workspace allows, against the
fp64 oracle with the bars of the other parity tests; and where cutting would not pay, whole items with no adding pass."""
import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc
from paper_2412_07894_amd import binding, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def names_of(run):
    binding.enable_kernel_timing(True)
    try:
        run()
        return [n for n, _ in binding.kernel_times()]
    finally:
        binding.enable_kernel_timing(False)


# one key tile of 16 steps; steps that q does not divide; a short tile behind a long one; parts bound by dQ; none where items fill the launch
@pytest.mark.parametrize("lens,hq,hkv,d,parts", [
    ([33], 8, 1, 128, True), ([256], 32, 8, 64, True), ([393, 307], 32, 8, 128, True), ([900], 2, 1, 64, True), ([1500], 8, 8, 128, True),
    ([1126, 374], 8, 8, 64, True), ([700], 32, 8, 128, True), ([64], 32, 8, 128, False), ([700], 32, 32, 64, False), ([640], 4, 4, 128, False)])
def test_parts_of_a_small_batch_match_the_oracle(lens, hq, hkv, d, parts):
    print(f"\n{lens} {hq}/{hkv} d = {d}", flush=True)
    T, scale = sum(lens), 1.0 / float(np.sqrt(d))
    cu, *host = wl.custom(lens, hq, hkv, d, "bf16", 83)
    q, k, v, do = (gu.to_dev(x, "bf16") for x in host)
    cu_d = torch.from_numpy(cu).cuda()
    o, lse = binding.varlen_attn_fwd(q, k, v, cu_d, max(lens), scale)
    rdq, rdk, rdv = orc.bwd(*host, cu, scale)
    full = binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 1)
    one = 2 * 4 * T * hkv * d
    for room in (0, 1, 2) if parts else (0,):         # the whole room, one part less of it, one more
        if full - room * one < one:
            break
        ws = torch.full((full - room * one,), 0xff, dtype=torch.uint8, device="cuda")        # (NaN in fp32)
        run = lambda: binding.varlen_attn_bwd(q, k, v, o, lse, do, cu_d, max(lens), scale, workspace=ws)
        try:
            names = names_of(run)
        except binding.HydError as e:                # less than the call itself needs
            assert room > 0 and e.code == 7          # HYD_ERR_WORKSPACE
            break
        assert "bwd_both_bf16" in names
        if room == 0:
            assert ("bwd_sum_parts" in names) == parts
        got, again = run(), run()
        for name, x, y, ref in zip(("dq", "dk", "dv"), got, again, (rdq, rdk, rdv)):
            assert torch.equal(x, y), name
            gu.check(name, gu.to_np(x), ref, "bf16")


# parts of the longest item: where the items alone nearly fill the launch, those that other launches take; else as fine as all begin at once
@pytest.mark.parametrize("lens,hq,hkv,d,least,most", [([4000], 8, 4, 64, 8, 8), ([7000], 4, 2, 128, 8, 8), ([14000], 2, 1, 128, 8, 8), ([5000], 4, 1, 128, 6, 7), ([3000], 8, 2, 64, 4, 6)])
def test_parts_by_the_room_of_the_launch(lens, hq, hkv, d, least, most):
    print(f"\n{lens} {hq}/{hkv} d = {d}", flush=True)
    T, scale = sum(lens), 1.0 / float(np.sqrt(d))
    cu, *host = wl.custom(lens, hq, hkv, d, "bf16", 89)
    q, k, v, do = (gu.to_dev(x, "bf16") for x in host)
    cu_d = torch.from_numpy(cu).cuda()
    o, lse = binding.varlen_attn_fwd(q, k, v, cu_d, max(lens), scale)
    ws = torch.full((binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 1),), 0xff, dtype=torch.uint8, device="cuda")
    run = lambda: binding.varlen_attn_bwd(q, k, v, o, lse, do, cu_d, max(lens), scale, workspace=ws)
    assert "bwd_both_bf16" in names_of(run)
    got = run()
    rec = binding.executed_items(ws, T, len(lens), hq, hkv, d, binding.HYD_BF16, 1, 0)[2]
    assert least <= rec[:, 5].max() <= most
    if T <= 4000:
        for name, x, ref in zip(("dq", "dk", "dv"), got, orc.bwd(*host, cu, scale)):
            gu.check(name, gu.to_np(x), ref, "bf16")
