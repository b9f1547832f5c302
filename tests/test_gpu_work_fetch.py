"""Work fetch of the persistent kernels around its special counts: fewer (item, head) pairs than
queues or workgroups, exactly as many, one more (the first claim through a cursor), queues of unequal
length (heads that do not divide over the eight queues), and items enough for several rounds."""
import pytest

from oracle import attn_oracle as orc
from paper_2412_07894_amd import workloads as wl
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,hq,hkv,dtype", [
    ([5], 1, 1, "bf16"),                         # one pair
    ([40] * 7, 1, 1, "bf16"),                    # fewer pairs than queues
    ([3] * 32, 8, 8, "bf16"),                    # 256 pairs: every workgroup has its fixed one
    ([3] * 33, 8, 8, "bf16"),                    # 264: the last eight are claimed
    ([3] * 51 + [70], 5, 5, "bf16"),             # striped queues of 35 and 30 pairs
    ([9] * 300 + [0, 700], 3, 1, "bf16"),        # several rounds, one long item list
    ([3] * 65, 4, 2, "fp32"),
    ([9] * 150 + [0, 300], 3, 1, "fp32"),
])
def test_counts_of_items_and_workgroups(lengths, hq, hkv, dtype):
    d = 64
    cu, q, k, v, do = wl.custom(lengths, hq, hkv, d, dtype, seed=95)
    scale = d ** -0.5
    got = gu.run_gpu(cu, q, k, v, do, dtype, scale)
    failures = []
    gu.check_all(got, q, k, v, do, cu, scale, dtype, failures, orc)
    assert not failures, "\n".join(failures)
