"""fp32 kernels on what unit-normal inputs never show: rows whose scores are strongly negative,
scores of -inf or below every finite mask value, tokens with infinities or NaN (which may reach their own
row and later ones, never an earlier one), and buffers that are only aligned to a float."""
import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc
from paper_2412_07894_amd import binding, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


def run(lengths, q, k, v, do, scale):
    cu = torch.from_numpy(wl.cu_seqlens(lengths)).cuda()
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (q, k, v, do)]
    o, lse = binding.varlen_attn_fwd(*dev[:3], cu, max(lengths), scale)
    dq, dk, dv = binding.varlen_attn_bwd(*dev[:3], o, lse, dev[3], cu, max(lengths), scale)
    return {n: gu.to_np(x) for n, x in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv))}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 33, 70, 160])
@pytest.mark.parametrize("low", [-80.0, -100.0, -300.0])
def test_last_row_with_strongly_negative_scores(low, L, d):
    """LSE of the last row near `low`: rows past a sequence that is no multiple of 32 long must not take part."""
    hq, hkv, scale = 4, 2, d ** -0.5
    cu, q, k, v, do = wl.custom([L, 40], hq, hkv, d, "fp32", seed=31)
    q[L - 1, :, :], k[:L] = 0.0, k[:L] * 0.1
    q[L - 1, :, 0], k[:L, :, 0] = low / scale, 1.0
    got = run([L, 40], q, k, v, do, scale)
    assert np.all(np.abs(got["lse"][:, L - 1] - low) < 0.1 * abs(low) + 10)
    o, lse = orc.fwd(q, k, v, cu, float(np.float32(scale)))
    ref = dict(zip(("dq", "dk", "dv"), orc.bwd(q, k, v, do, cu, float(np.float32(scale)))))
    for name, r in {"o": o, "lse": lse, **ref}.items():
        max_abs, rel = gu.errors(got[name], r)
        print(f"{name}: max-abs {max_abs:.2e} rel-L2 {rel:.2e}", flush=True)
        # a score of size |low| is a sum of d products: 2^-24 |low| sqrt(d) of absolute error in the exponent of P
        assert np.all(np.isfinite(got[name])) and rel <= 1e-5 + 2.0 ** -23 * abs(low) * np.sqrt(d), name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("at", [20, 40, 130])
def test_a_score_of_minus_infinity_is_a_probability_of_zero(at, d):
    """q . k overflows to -inf for one key: that key is not attended to."""
    L, hq, hkv, scale = 200, 2, 1, d ** -0.5
    cu, q, k, v, do = wl.custom([L], hq, hkv, d, "fp32", seed=32)
    q[:, :, 0], k[:, :, 0] = 1e30, 0.0
    k[at, :, 0] = -1e30
    got = run([L], q, k, v, do, scale)
    o, lse = orc.fwd(q, k, v, cu, scale)
    dq, dk, dv = orc.bwd(q, k, v, do, cu, scale)
    for name, x, ref in (("o", got["o"], o), ("lse", got["lse"], lse), ("dq", got["dq"][:, :, 1:], dq[:, :, 1:]), ("dv", got["dv"], dv)):
        assert np.all(np.isfinite(x)) and gu.errors(x, ref)[1] <= 1e-5, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("score", [-1e31, -1e38])
def test_scores_below_any_mask_value(score, d):
    """All scores equal and hugely negative: every row is the mean of the V up to it."""
    L, hq, hkv = 100, 2, 1
    cu, q, k, v, do = wl.custom([L], hq, hkv, d, "fp32", seed=33)
    q[:], k[:] = 0.0, 0.0
    q[:, :, 0], k[:, :, 0] = score, 1.0
    dev = [torch.from_numpy(x).cuda() for x in (q, k, v)]
    o, lse = binding.varlen_attn_fwd(*dev, torch.from_numpy(cu).cuda(), L, 1.0)
    ro, rlse = orc.fwd(q, k, v, cu, 1.0)
    assert gu.errors(gu.to_np(o), ro)[1] <= 1e-5 and gu.errors(gu.to_np(lse), rlse)[1] <= 1e-5


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("at", [5, 31, 32, 70, 149])
def test_a_bad_token_stays_out_of_earlier_rows(at, bad, d):
    """Row `at` of one tensor at a time holds `bad`.  O, LSE and dQ of earlier rows depend on Q, K and V up to
    themselves, dK and dV of later keys on rows of Q and dO from themselves on: they are what they are without it."""
    L, hq, hkv, scale = 150, 4, 2, d ** -0.5
    _, q, k, v, do = wl.custom([L], hq, hkv, d, "fp32", seed=34)
    clean = run([L], q, k, v, do, scale)
    for name in ("q", "k", "v", "do"):
        x = {"q": q.copy(), "k": k.copy(), "v": v.copy(), "do": do.copy()}
        x[name][at, :, 3] = bad
        got = run([L], x["q"], x["k"], x["v"], x["do"], scale)
        parts = [("o", got["o"][:at], clean["o"][:at]), ("lse", got["lse"][:, :at], clean["lse"][:, :at]), ("dq", got["dq"][:at], clean["dq"][:at])]
        if name in ("q", "do"):                            # K and V of one key reach all rows from it on, and with them every key
            parts += [(out, got[out][at + 1:], clean[out][at + 1:]) for out in ("dk", "dv")]
        for out, a, b in parts:                            # (the sums of one block in another order: no more than the kernels' bar)
            assert np.all(np.isfinite(a)) and (a.size == 0 or gu.errors(a, b)[1] <= 1e-6), (name, out)


@pytest.mark.parametrize("d", [64, 128])
def test_buffers_aligned_to_one_float(d):
    """Tensors that start at any float of a larger allocation, as a slice of a flat parameter buffer does."""
    lengths, hq, hkv = [77, 130], 4, 2
    cu, q, k, v, do = wl.custom(lengths, hq, hkv, d, "fp32", seed=35)
    ref = run(lengths, q, k, v, do, d ** -0.5)
    cu_d = torch.from_numpy(cu).cuda()

    def odd(x, shift):
        buf = torch.zeros(x.size + 8, dtype=torch.float32, device="cuda")
        view = buf[shift:shift + x.size].view(x.shape)
        view.copy_(torch.from_numpy(np.ascontiguousarray(x)))
        assert view.data_ptr() % 16 == 4 * shift
        return view
    for shift in (1, 2, 3):
        dq_, dk_, dv_, o_ = (odd(np.zeros_like(x), shift) for x in (q, k, v, q))
        qs, ks, vs, dos = (odd(x, shift) for x in (q, k, v, do))
        o, lse = binding.varlen_attn_fwd(qs, ks, vs, cu_d, max(lengths), d ** -0.5, out=o_)
        binding.varlen_attn_bwd(qs, ks, vs, o, lse, dos, cu_d, max(lengths), d ** -0.5, dq=dq_, dk=dk_, dv=dv_)
        for name, x in (("o", o), ("lse", lse), ("dq", dq_), ("dk", dk_), ("dv", dv_)):
            assert np.array_equal(gu.to_np(x), ref[name]), (shift, name)
