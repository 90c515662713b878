"""The local sort that ranks elements in bins (k_local_rank): segment sizes at
the edges of its workgroup shapes, and key forms for each way its 32-bit words
can fail to tell elements apart (equal words, equal keys, too crowded bins),
bit-exact against the oracle's per-array sort.  All results are whole numbers:
the tolerance is zero."""
import numpy as np
import pytest

from gen import gen
from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import gpu_segmented, gpu_sort, same_bits

pytestmark = pytest.mark.gpu

# 64 x 4, 256 x 4, 512 x 8, 512 x 12, 1024 x 8 and 1024 x 12 elements, and
# the first element of a second round of the shapes' threads
EDGES = [65, 255, 256, 257, 511, 513, 1023, 1024, 1025, 4095, 4096, 4097, 6143, 6144, 6145, 8191, 8192, 8193, 12287,
         12288, 2, 1]


def _keys(form, kt, n, rng):
    dt = np.uint64 if kt == "u64" else np.uint32
    bits = 64 if kt == "u64" else 32
    r = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    if form == "equal_words":  # wide range; many keys differ in their low bits only
        k = (rng.integers(0, 64, n, dtype=np.uint64) << np.uint64(bits - 8)) + (r & np.uint64(0xFFFFF if bits == 64 else 0xFF))
    elif form == "wide_dup":  # 40 distinct keys over the whole range: equal keys in every bin
        pool = rng.integers(0, 1 << 63, 40, dtype=np.uint64) * np.uint64(2) + np.uint64(1)
        k = (pool >> np.uint64(64 - bits))[rng.integers(0, 40, n)]
    elif form == "extremes":  # the type's smallest and largest keys among random ones
        k = r >> np.uint64(64 - bits)
        k[rng.random(n) < 0.3] = 0
        k[rng.random(n) < 0.3] = (1 << bits) - 1
    elif form == "halves":  # two clusters far apart: crowded bins
        k = (r & np.uint64(3)) + (rng.integers(0, 2, n, dtype=np.uint64) << np.uint64(bits - 1))
    else:  # "straddle": two neighbouring keys, each in few positions' reach
        k = np.where(np.arange(n) < n // 3, np.uint64(8), np.uint64(7)).astype(np.uint64)
    return k.astype(dt).view(np.float32) if kt == "f32" else k.astype(dt)


@pytest.mark.parametrize("kt", ["u64", "u32", "f32"])
@pytest.mark.parametrize("form", ["equal_words", "wide_dup", "extremes", "halves", "straddle"])
@pytest.mark.parametrize("with_payload", [False, True])
def test_segments_at_shape_edges(kt, form, with_payload):
    rng = np.random.default_rng(len(form) * 7 + len(kt))
    keys = np.concatenate([_keys(form, kt, n, rng) for n in EDGES])
    off = np.concatenate([[0], np.cumsum(EDGES)]).astype(np.uint64)
    pay = rng.integers(0, 1 << 32, keys.size, dtype=np.uint64).astype(np.uint32) if with_payload else None
    ko, po, plo, _ = gpu_segmented(keys, off, pay)
    ek, ep, epl = O.segmented(keys, off, pay)
    assert same_bits(ko, ek) and np.array_equal(po, ep)
    if with_payload:
        assert np.array_equal(plo, epl)


@pytest.mark.parametrize("kt", ["u64", "u32"])
@pytest.mark.parametrize("distinct", [1 << 12, 1 << 16])
def test_buckets_with_equal_keys(kt, distinct):
    """Final buckets of a split sort whose keys repeat over a wide range, in
    any order of positions, with and without the permutation."""
    rng = np.random.default_rng(distinct)
    pool = np.unique(rng.integers(0, 1 << (63 if kt == "u64" else 32), distinct, dtype=np.uint64))
    x = pool[rng.integers(0, pool.size, 3_000_001)].astype(np.uint64 if kt == "u64" else np.uint32)
    ek, ep, _ = O.sort(x, threads=8)
    ko, po = gpu_sort(x)
    assert same_bits(ko, ek) and np.array_equal(po, ep)
    ko, po = gpu_sort(x, with_perm=False)
    assert po is None and same_bits(ko, ek)


def test_many_segments_per_workgroup():
    """More segments than workgroups in every shape, of all sizes: a workgroup
    loads its next segment while it writes one out, across class borders and
    past segments it hands over."""
    rng = np.random.default_rng(3)
    sizes = rng.integers(1, 8193, 9000).astype(np.uint64)
    keys, pay, off = gen.segmented("u32", sizes, gen.pick_dists(sizes.size, ["uniform", "zero", "deterdupl"], seed=4),
                                   seed=6)
    half = rng.random(keys.size) < 0.5
    for s in range(0, sizes.size, 11):  # crowded bins: left to the merge sort
        a, b = int(off[s]), int(off[s + 1])
        keys[a:b] = np.where(half[a:b], keys[a:b] & 7, 0xFFFFFF00 + (keys[a:b] & 7)).astype(np.uint32)
    ko, po, plo, _ = gpu_segmented(keys, off, pay)
    ek, ep, epl = O.segmented(keys, off, pay)
    assert same_bits(ko, ek) and np.array_equal(po, ep) and np.array_equal(plo, epl)


@pytest.mark.parametrize("kt", ["u64", "u32", "f32"])
@pytest.mark.parametrize("form", ["wide_dup", "halves", "straddle"])
@pytest.mark.parametrize("n", [200, 1000, 1025, 4096, 4097, 8192, 8193, 12288])
def test_direct_calls(kt, form, n):
    """Plain calls of one workgroup, whose crowded bins are merge sorted in the
    same launch (up to 8192 keys) or in the next."""
    x = _keys(form, kt, n, np.random.default_rng(n))
    ek, ep, _ = O.sort(x)
    ko, po = gpu_sort(x)
    assert same_bits(ko, ek) and np.array_equal(po, ep)
