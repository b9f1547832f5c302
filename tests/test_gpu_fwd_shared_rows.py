"""Forward items of 64 rows whose waves share them (head dimension 128, few items): bit for bit what whole tiles give, with
and without an item list, and against fp64 where the reference of a row has to move."""
import numpy as np
import pytest
import torch

from paper_2412_07894_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu
D = 128


def forward(q, k, v, lens, scale, rope_base=None):
    return binding.varlen_attn_fwd(q, k, v, torch.from_numpy(wl.cu_seqlens(lens)).cuda(), max(lens), scale, rope_base=rope_base)


def inputs(T, hq, hkv, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.randn((T, h, D), device="cuda", generator=g).to(torch.bfloat16) for h in (hq, hkv, hkv)]


def path(q, k, v, lens, scale, rope_base=None):
    """O, LSE, the rows of a tile that the forward took, and whether it took them from a list."""
    T, hq, hkv, d = sum(lens), q.shape[1], k.shape[1], q.shape[2]
    ws = torch.empty(binding.workspace_bytes(T, len(lens), hq, hkv, d, binding.HYD_BF16, 0), dtype=torch.uint8, device="cuda")
    binding.enable_kernel_timing(True)
    try:
        o, lse = binding.varlen_attn_fwd(q, k, v, torch.from_numpy(wl.cu_seqlens(lens)).cuda(), max(lens), scale, workspace=ws, rope_base=rope_base)
        names = [n for n, _ in binding.kernel_times()]
    finally:
        binding.enable_kernel_timing(False)
    return o, lse, binding.executed_items(ws, T, len(lens), hq, hkv, d, binding.HYD_BF16, 0, 0)[0], "schedule_prelude" in names


# each sequence a workgroup's own; the same of a second round; a list because there are more sequences than such a launch takes, or because the items are long
CASES = [([1, 63, 64, 65, 127, 128, 129, 191, 193], 4, 2, False), ([1100] * 9, 2, 1, False), ([28] * 256 + [1100], 1, 1, True), ([6200], 3, 3, True)]


@pytest.mark.parametrize("lens,hq,hkv,listed", CASES)
@pytest.mark.parametrize("rope_base", [None, 1e4])
def test_same_bits_as_whole_tiles(lens, hq, hkv, listed, rope_base):
    T, copies = sum(lens), 1 + 12000 // (len(lens) * hq) if max(lens) < 1000 else 48
    q, k, v = inputs(T, hq, hkv, 61)
    print(f"\n{len(lens)} sequences, {T} tokens, {hq}/{hkv}, rope {rope_base}", flush=True)
    o, lse, tile, from_list = path(q, k, v, lens, D ** -0.5, rope_base)
    assert (tile, from_list) == (64, listed), "the sizes are meant to take the form"
    o2, lse2, tile, _ = path(*(t.repeat(copies, 1, 1) for t in (q, k, v)), lens * copies, D ** -0.5, rope_base)
    assert tile == 256
    assert bool(torch.isfinite(o.float()).all())
    assert torch.equal(o, o2[-T:]) and torch.equal(lse, lse2[:, -T:])


@pytest.mark.parametrize("lens,hq,tile", [([256], 8, 64), ([4000], 8, 64), ([25600], 1, 64), ([2880], 10, 128), ([6528], 5, 128), ([6000], 8, 128), ([2900], 10, 128)])
def test_form_of_one_sequence(lens, hq, tile):
    """64 rows per item where all or nearly all items begin at once; from a list only where an XCD keeps to few heads."""
    q, k, v = inputs(sum(lens), hq, hq, 71)
    assert path(q, k, v, lens, D ** -0.5)[2] == tile


# (tile without, with rotary positions)
@pytest.mark.parametrize("lens,hq,tile,rotary", [([81] * 12, 8, 64, 64), ([81] * 19, 8, 128, 128), ([600] * 11, 3, 128, 128), ([900] * 8, 2, 64, 64), ([900] * 10, 2, 64, 128), ([1100] * 9, 2, 64, 64),
                                                 ([2712] + [1926] * 4, 3, 128, 128), ([3200, 800], 8, 64, 64)])
def test_form_where_items_come_second(lens, hq, tile, rotary):
    """Items of 64 rows that do not all begin at once only where sequences are long; rotary positions make an item dearer."""
    q, k, v = inputs(sum(lens), hq, hq, 73)
    assert path(q, k, v, lens, D ** -0.5)[2] == tile and path(q, k, v, lens, D ** -0.5, 1e4)[2] == rotary


@pytest.mark.parametrize("scale", [D ** -0.5, -D ** -0.5])
@pytest.mark.parametrize("gain", [1.0, 24.0])
def test_rows_whose_reference_moves(gain, scale):
    """Keys that grow along the sequence, so that the largest score of a row keeps rising (or, with a negative scale,
    falling).  P is rounded to bf16 and its sum is taken of the rounded values: |dO| <= 2 * 2^-9 max|V|, and 2^-9 |O| more for the
    store; scores of up to 2^11 in fp32 (fewer than 2^3 roundings of 2^-24 each) move P by 2^-9."""
    lens, hq = [513, 130, 700], 4
    T = sum(lens)
    q, k, v = inputs(T, hq, hq, 67)
    ramp = torch.cat([torch.linspace(0.1, 1.0, n) for n in lens]).cuda().reshape(T, 1, 1) * gain
    k = (k.float() * ramp).to(torch.bfloat16)
    print(f"\ngain {gain} scale {scale}", flush=True)
    o, lse = forward(q, k, v, lens, scale)
    qd, kd, vd = (t.double().cpu().numpy() for t in (q, k, v))
    row = 0
    for n in lens:
        for h in range(hq):
            s = qd[row:row + n, h] @ kd[row:row + n, h].T * scale
            s[np.triu_indices(n, 1)] = -np.inf
            m = s.max(1, keepdims=True)
            p = np.exp(s - m)
            l = p.sum(1, keepdims=True)
            ref, top = (p / l) @ vd[row:row + n, h], np.abs(vd[row:row + n, h]).max()
            assert np.abs(o[row:row + n, h].double().cpu().numpy() - ref).max() <= 2.0 ** -6 * top
            assert np.abs(lse[h, row:row + n].double().cpu().numpy() - (m + np.log(l))[:, 0]).max() <= 2.0 ** -8
        row += n
