"""The backward's preparation pass splits the tokens over its workgroups by batch size: one token per
workgroup up to 1024 tokens, a ragged last block, partial maxima of |dO| whose count is no multiple
of four.  The largest |dO| of the tensor sits in the last row, the only one its workgroup sees, and
is so much larger that dO would leave the range of fp16 if that workgroup's maximum got lost.

Tolerance: the gradients are linear in dO, so the rel-L2 bar holds whatever its scale; the max-abs bar
is for dO of order one, which the rows of dQ before the last one are."""
import numpy as np
import pytest

from oracle import attn_oracle as orc
from paper_2412_07894_amd import workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,hq,hkv", [
    ([1], 2, 1),
    ([1000, 23], 4, 2),                  # one token per workgroup
    ([1500, 1499, 0, 2], 2, 1),          # three per workgroup, a last block of one token (its dK would be zero in a sequence of its own)
    ([2100, 1030, 993], 3, 3),           # five per workgroup
])
def test_preparation_pass_splits(lengths, hq, hkv, d):
    cu, q, k, v, do = wl.custom(lengths, hq, hkv, d, "bf16", seed=91)
    do[-1] *= np.float32(2.0 ** 20)
    scale = d ** -0.5
    got = gu.run_gpu(cu, q, k, v, do, "bf16", scale)
    gq, gk, gv = orc.bwd_given(q, k, v, do, got["o"].astype(np.float32), got["lse"].astype(np.float32), cu, scale)
    for name, ref in (("dq", gq), ("dk", gk), ("dv", gv)):
        max_abs, rel = gu.errors(got[name], ref)
        print(f"{name}: rel-L2 {rel:.3e}", flush=True)
        assert np.all(np.isfinite(got[name])) and rel <= gu.TOL["bf16"][1], name
    if cu[-1] > 1:
        gu.check("dq before the last row", got["dq"][:-1], gq[:-1], "bf16")
