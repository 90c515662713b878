"""Final segments above the LDS capacity (k_local_rare): one chunk or many per
segment, ties, payloads, outputs left out, and segments that must not touch
the other buffer because segments of it were handed over; bit-exact against the
oracle (whole numbers, zero tolerance).  They are sorted by as many workgroups as
there are segments."""
import numpy as np
import pytest
import torch

from gen import gen
from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import banner, dev, gpu_segmented, gpu_sort, host, same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kt", ["u64", "u32", "f32"])
@pytest.mark.parametrize("dist", ["uniform", "zero", "deterdupl"])
@pytest.mark.parametrize("tune,n", [(dict(oversample=1), 3_000_001), (dict(max_levels=1), (1 << 24) + 3),
                                    (dict(force_fallback=1), 400_003)])
def test_plain_oversize_buckets(kt, dist, tune, n):
    """Buckets of up to a few times the capacity (one sample per bucket), of
    three chunks each (one level where two are planned), and of less than the
    capacity (the switch that sends all of them this way)."""
    x = gen.keys(kt, dist, n, seed=n % 97)
    ek, ep, _ = O.sort(x, threads=8)
    kty = {"u64": R.U64, "u32": R.U32, "f32": R.F32}[kt]
    with R.tuned(**tune):
        ws = torch.empty(R.plain_workspace_bytes(kty, n), dtype=torch.uint8, device="cuda")
        banner("oversize buckets %s %s %s n=%d" % (kt, dist, tune, n))
        ko, po = R.sort(dev(x), workspace=ws)
        st = R.stats(ws)
        assert st["status"] == 0 and st["oversize"] > 0
        assert same_bits(host(ko), ek) and np.array_equal(host(po), ep)
        ko, po = gpu_sort(x, with_perm=False)
        assert po is None and same_bits(ko, ek)


@pytest.mark.parametrize("kt", ["u64", "u32"])
@pytest.mark.parametrize("with_perm", [True, False])
@pytest.mark.parametrize("crowded", [False, True])
def test_segmented_oversize_buckets(kt, with_perm, crowded):
    """Segments split once and twice in one call, with a payload and one sample
    per bucket.  With crowded keys in the former, buckets that lie in the
    buffer the oversize ones of the latter would write to are handed over."""
    sizes = np.array([1_000_000, 6_000_000, 90_000, 700], dtype=np.uint64)
    keys, pay, off = gen.segmented(kt, sizes, ["uniform", "uniform", "zero", "uniform"], seed=23)
    if crowded:  # two clusters far apart in every bucket that holds the middle
        rng = np.random.default_rng(1)
        bits = 64 if kt == "u64" else 32
        low = rng.integers(0, 1 << 12, 1_000_000, dtype=np.uint64)
        keys[:1_000_000] = np.where(rng.random(1_000_000) < 0.995, low, low << np.uint64(bits - 13)).astype(keys.dtype)
    ek, ep, epl = O.segmented(keys, off, pay)
    with R.tuned(oversample=1):
        ko, po, plo, _ = gpu_segmented(keys, off, pay, with_perm=with_perm)
    assert same_bits(ko, ek) and np.array_equal(plo, epl)
    if with_perm:
        assert np.array_equal(po, ep)


def test_oversize_segments_are_sorted_side_by_side():
    """A sort whose 1024 buckets all go this way takes a few times as long as
    the ordinary one (2.3 times; 400 when one workgroup sorted them all); the
    bound leaves a factor of eight."""
    x = dev(gen.keys("u64", "uniform", 6_000_001, seed=3))

    def ms():
        R.sort(x)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            R.sort(x)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 3

    banner("time of an ordinary sort and of one by the fallback")
    ordinary = ms()
    with R.tuned(force_fallback=1):
        fallback = ms()
    assert fallback < 20 * ordinary, (ordinary, fallback)
