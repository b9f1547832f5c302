"""The forward takes its softmax reference from a row's first tile of keys.  Scores that rise later
must move it exactly: by a little (no action), by more than 2^24 in the row sum (O and l are scaled
back), by so much that a probability overflows (the item is repeated with the true row maxima), in
any tile, also the diagonal one, and next to rows and heads where nothing happens."""
import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc
from paper_2412_07894_amd import binding, workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("gain", [3.0, 12.0, 60.0])      # largest score 12, 50, 250 (natural log units)
@pytest.mark.parametrize("first_key", [40, 64, 250, 690])
def test_scores_that_rise_after_the_first_tile(gain, first_key, d):
    lengths, hq, hkv = [700, 90, 300], 4, 2
    cu, q, k, v, do = wl.custom(lengths, hq, hkv, d, "bf16", seed=81)
    for s, L in enumerate(lengths):                       # KV head 0 only: heads 2 and 3 stay ordinary
        k[cu[s] + first_key:cu[s] + L, 0] *= gain
    k = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(k))
    scale = d ** -0.5
    got = gu.run_gpu(cu, q, k, v, do, "bf16", scale)
    o, lse = orc.fwd(q, k, v, cu, scale)
    gu.check("o", got["o"], o, "bf16")
    # LSE is as large as the scores here: fp32 sums of d products of that size
    tol = max(2e-2, 2.0 ** -23 * np.sqrt(d) * np.max(np.abs(lse)) * 4)
    assert np.max(np.abs(got["lse"] - lse)) <= tol


def forward(lengths, q, k, v, scale):
    """Forward over bf16-exact float32 inputs: O and LSE as float64, then the oracle's."""
    cu = wl.cu_seqlens(lengths)
    for x in (q, k, v):
        assert np.array_equal(x, wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(x))), "inputs are bf16 values"
    dev = [gu.to_dev(x, "bf16") for x in (q, k, v)]
    o, lse = binding.varlen_attn_fwd(*dev, torch.from_numpy(cu).cuda(), max(lengths), scale)
    return gu.to_np(o), gu.to_np(lse), *orc.fwd(q, k, v, cu, float(np.float32(scale)))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("key,L", [(100, 128), (100, 192), (100, 700), (300, 700)])     # in the row's last tile, in an earlier one
@pytest.mark.parametrize("rise", [100.0, 126.0, 126.5, 127.0, 127.5, 127.99, 128.5, 200.0])
def test_one_key_far_above_the_first_tile(rise, key, L, d):
    """One key scores `rise` (log2 units) above all others, which score 0, with V of at most 0.5: the row sum runs up
    to the largest finite values and O with it.  The row is that key's V from then on."""
    hq, hkv, scale = 4, 2, d ** -0.5
    rng = np.random.default_rng(5)
    q, k = np.zeros((L, hq, d), np.float32), np.zeros((L, hkv, d), np.float32)
    v = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(rng.uniform(-0.5, 0.5, (L, hkv, d)).astype(np.float32)))
    q[:, :, :3] = 16.0
    want = rise / (16.0 * scale * np.log2(np.e))
    for c in range(3):                                     # three bf16 pieces: the score is right to 2^-16
        k[key, 0, c] = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(np.array([want], np.float32)))[0]
        want -= float(k[key, 0, c])
    o, lse, ro, rlse = forward([L], q, k, v, scale)
    assert abs(rlse[0, key] * np.log2(np.e) - rise) < 2e-3
    gu.check("o", o, ro, "bf16")
    assert np.max(np.abs(lse - rlse)) <= 2e-2


@pytest.mark.parametrize("d", [64, 128])
def test_scores_beyond_the_integers_of_a_float(d):
    """Scores of 2^26 (log2 units), where a float holds every eighth integer: three keys 24 above the first tile with
    V = 0.5, three more of the same score in the tile after with V = -0.5, so O is 0 from there on.  The reference can
    only move by what it holds, and O and l have to be scaled by exactly that."""
    L, hq, hkv = 256, 2, 1
    scale = float(np.float32(np.log(2.0)))
    q, k = np.zeros((L, hq, d), np.float32), np.zeros((L, hkv, d), np.float32)
    v = np.zeros((L, hkv, d), np.float32)
    q[:, :, 0], q[:, :, 1] = 2.0 ** 13, 8.0
    k[:, 0, 0] = 2.0 ** 13
    for at, val in ((64, 0.5), (128, -0.5)):
        k[at:at + 3, 0, 1] = 3.0
        v[at:at + 3] = val
    o, _, ro, _ = forward([L], q, k, v, scale)
    assert np.max(np.abs(o[131:] - ro[131:])) <= 2e-2 and np.max(np.abs(ro[131:])) < 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("key,L", [(100, 128), (100, 300), (299, 300)])
def test_large_values_times_a_large_probability(key, L, d):
    """V of 2^105 and one key 23.5 (log2 units) above all others: O passes the largest float while the row sum
    stays below the limit from which it is scaled back.  O itself is no larger than V."""
    hq, hkv, scale = 4, 2, d ** -0.5
    rng = np.random.default_rng(6)
    q, k = np.zeros((L, hq, d), np.float32), np.zeros((L, hkv, d), np.float32)
    unit = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(rng.uniform(0.75, 1.0, (L, hkv, d)).astype(np.float32)))
    q[:, :, 0] = 16.0
    k[key, 0, 0] = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(np.array([23.5 / (16.0 * scale * np.log2(np.e))], np.float32)))[0]
    o, lse, ro, rlse = forward([L], q, k, unit * np.float32(2.0 ** 105), scale)
    gu.check("o / 2^105", o * 2.0 ** -105, ro * 2.0 ** -105, "bf16")
    assert np.max(np.abs(lse - rlse)) <= 2e-2
