"""GPU parity of the fp32 kernels at the sizes where their tiling can go wrong: 32-row blocks (a
wave), 64-row items, 128-row streamed tiles split over four waves, lengths on both sides of each.

Tolerance.  rel-L2 1e-5 as everywhere; max-abs 1e-5 as long as sums are short.  A gradient of a key is
a running fp32 sum of n = (query rows) x (heads of the group) terms, a quarter of them in each of
four waves: every addition rounds by at most u = 2^-24 of a partial sum of at most max|ref| (uniformly
distributed, standard deviation u max|ref| / sqrt(3)), so four standard deviations of n / 4
independent roundings are 4 / sqrt(3) u sqrt(n / 4) max|ref|; that is allowed where it exceeds 1e-5."""
import numpy as np
import pytest

from oracle import attn_oracle as orc
from paper_2412_07894_amd import workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,hq,hkv", [
    ([1, 31, 32, 33, 63, 64, 65, 0, 96, 97], 2, 2),         # blocks and items
    ([127, 128, 129, 191, 193, 257], 4, 2),                 # streamed tiles; grouped heads
    ([520], 8, 1),                                          # several tiles, the whole group in one item
])
def test_fp32_tile_edges(lengths, hq, hkv, d):
    cu, q, k, v, do = wl.custom(lengths, hq, hkv, d, "fp32", seed=71)
    scale = d ** -0.5
    got = gu.run_gpu(cu, q, k, v, do, "fp32", scale)
    o, lse = orc.fwd(q, k, v, cu, scale)
    dq, dk, dv = orc.bwd(q, k, v, do, cu, scale)
    for name, ref in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        n = max(lengths) * (hq // hkv if name in ("dk", "dv") else 1)
        tol = max(1e-5, 4 / np.sqrt(3) * 2.0 ** -24 * np.sqrt(n / 4) * np.max(np.abs(ref)))
        max_abs, rel = gu.errors(got[name], ref)
        print(f"{name}: max-abs {max_abs:.3e} (tol {tol:.1e})  rel-L2 {rel:.3e}", flush=True)
        assert np.all(np.isfinite(got[name])) and max_abs <= tol and rel <= 1e-5, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,hq,hkv", [
    ([8, 1, 0, 7, 5, 8, 3, 2], 4, 2),                       # nothing but short sequences
    ([8, 9, 1, 40, 7, 16], 8, 2),                           # on both sides of the limit
    ([1] * 300, 2, 2),                                      # more items than workgroups
])
def test_fp32_short_sequences(lengths, hq, hkv, d):
    cu, q, k, v, do = wl.custom(lengths, hq, hkv, d, "fp32", seed=72)
    scale = d ** -0.5
    got = gu.run_gpu(cu, q, k, v, do, "fp32", scale)
    o, lse = orc.fwd(q, k, v, cu, scale)
    for name, ref in zip(("o", "lse", "dq", "dk", "dv"), (o, lse) + tuple(orc.bwd(q, k, v, do, cu, scale))):
        max_abs, rel = gu.errors(got[name], ref)
        print(f"{name}: max-abs {max_abs:.3e} rel-L2 {rel:.3e}", flush=True)
        assert np.all(np.isfinite(got[name])) and max_abs <= 1e-5 and rel <= 1e-5, name
