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


# each sequence a workgroup's own; more sequences than such a launch takes; a list because the items are long
CASES = [([1, 63, 64, 65, 127, 128, 129, 191, 193], 4, 2), ([1] * 257, 1, 1), ([2] * 250 + [300] * 8, 1, 1), ([6200], 4, 4)]


@pytest.mark.parametrize("lens,hq,hkv", CASES)
@pytest.mark.parametrize("rope_base", [None, 1e4])
def test_same_bits_as_whole_tiles(lens, hq, hkv, rope_base):
    T, copies = sum(lens), 1 + 4000 // (len(lens) * hq) if max(lens) < 1000 else 24
    q, k, v = inputs(T, hq, hkv, 61)
    print(f"\n{len(lens)} sequences, {T} tokens, {hq}/{hkv}, rope {rope_base}", flush=True)
    o, lse = forward(q, k, v, lens, D ** -0.5, rope_base)
    o2, lse2 = forward(*(t.repeat(copies, 1, 1) for t in (q, k, v)), lens * copies, D ** -0.5, rope_base)
    assert bool(torch.isfinite(o.float()).all())
    assert torch.equal(o, o2[-T:]) and torch.equal(lse, lse2[:, -T:])


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
