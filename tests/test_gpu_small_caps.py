"""Single-level plain sorts under a reduced LDS capacity: all their buckets,
however short, go to the list of the one size class that holds the capacity.
Bit-exact against the oracle (whole numbers, zero tolerance), and no list may
overflow (the workspace status)."""
import numpy as np
import pytest
import torch

from gen import gen
from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import banner, dev, host, same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [64, 100, 256, 512, 1000, 1024, 2048, 3072, 4096, 5000, 6144, 8192])
@pytest.mark.parametrize("kt", ["u64", "u32"])
def test_one_level_plain_sorts_fill_one_class(cap, kt):
    """Sizes just above the capacity, with twice as many buckets as the target
    needs, at the most buckets of one level, and one between."""
    target = max(64, min(6144, cap // 2))
    for n in (cap + 1, 256 * target + 1, 512 * target, 16 * target + 777):
        x = gen.keys(kt, "uniform", n, seed=n % 1000)
        ek, ep, _ = O.sort(x, threads=8)
        with R.tuned(cap=cap):
            ws = torch.empty(R.plain_workspace_bytes(R.U64 if kt == "u64" else R.U32, n), dtype=torch.uint8,
                             device="cuda")
            banner("one-level plain sort cap=%d n=%d %s" % (cap, n, kt))
            ko, po = R.sort(dev(x), workspace=ws)
            st = R.stats(ws)
        assert st["status"] == 0 and st["levels"] == 1
        assert same_bits(host(ko), ek) and np.array_equal(host(po), ep)
