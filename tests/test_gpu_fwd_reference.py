"""The forward takes its softmax reference from a row's first tile of keys.  Scores that rise later
must move it exactly: by a little (no action), by more than 2^24 in the row sum (O and l are scaled
back), by so much that a probability overflows (the item is repeated with the true row maxima), in
any tile, also the diagonal one, and next to rows and heads where nothing happens."""
import numpy as np
import pytest

from oracle import attn_oracle as orc
from paper_2412_07894_amd import workloads as wl
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
