"""The split levels (tiles sorted by bucket and written back as one piece,
buckets read back as their runs): tile and level edges, buckets whose elements
lie in more tiles than a workgroup has threads, payloads through several
levels; bit-exact against the oracle (whole numbers, zero tolerance)."""
import numpy as np
import pytest

from gen import gen
from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import gpu_segmented, gpu_sort, same_bits

pytestmark = pytest.mark.gpu


def _check(x, threads=8):
    ek, ep, _ = O.sort(x, threads=threads)
    ko, po = gpu_sort(x)
    assert same_bits(ko, ek) and np.array_equal(po, ep)


@pytest.mark.parametrize("kt", ["u64", "u32"])
@pytest.mark.parametrize("n", [4096 * 4, 4096 * 4 + 1, 4096 * 5 - 1, 64 * 4096 + 63, 3145729, (1 << 23) - 1, 1 << 23,
                               (1 << 23) + 8191])
def test_tile_and_level_edges(kt, n):
    _check(gen.keys(kt, "uniform", n, seed=n))


@pytest.mark.parametrize("kt", ["u64", "f32"])
@pytest.mark.parametrize("n,tile_log2", [((1 << 22) + 5, 12), ((1 << 24) + 5, 13)])
@pytest.mark.parametrize("thin", [200, 3000])
def test_buckets_strewn_over_more_tiles_than_threads(kt, n, tile_log2, thin):
    """In the first three quarters one key in `thin` is small, in the last all
    are: the first elements of the buckets of small keys lie in more tiles than
    a workgroup has threads, a few or none in each."""
    rng = np.random.default_rng(thin)
    k = rng.random(n)
    small = (np.arange(n) >= 3 * n // 4) | (rng.random(n) < 1.0 / thin)
    k = np.where(small, k * 0.001, 0.5 + 0.5 * k)
    x = k.astype(np.float32) if kt == "f32" else (k * float(1 << 62)).astype(np.uint64)
    with R.tuned(tile_log2=tile_log2):
        _check(x)


@pytest.mark.parametrize("kt", ["u64", "u32"])
@pytest.mark.parametrize("cap", [256, 12288])
def test_payload_through_levels(kt, cap):
    """Segments split by no, one, two or three levels in one call, all with a
    payload; the local sorts of early levels run before a later level reuses
    their buffer."""
    sizes = np.array([5, 700000, 250, 0, 3400000, 257, 64, 13000, 90000, 300], dtype=np.uint64)
    keys, pay, off = gen.segmented(kt, sizes, ["uniform", "deterdupl", "zero", "zero", "gaussian", "uniform", "reverse",
                                               "uniform", "zero", "uniform"], seed=17)
    with R.tuned(cap=cap):
        ko, po, plo, _ = gpu_segmented(keys, off, pay)
    ek, ep, epl = O.segmented(keys, off, pay)
    assert same_bits(ko, ek) and np.array_equal(po, ep) and np.array_equal(plo, epl)


@pytest.mark.parametrize("kt", ["u64", "u32"])
def test_oversize_buckets_of_several_segments(kt):
    """One level only: many buckets exceed the LDS sort and are merge sorted
    through the buffers, next to segments that need no level."""
    sizes = np.array([400000, 100, 900000, 5000, 300000], dtype=np.uint64)
    keys, pay, off = gen.segmented(kt, sizes, ["uniform", "zero", "deterdupl", "uniform", "reverse"], seed=9)
    with R.tuned(max_levels=1, cap=1024, oversample=1, target=512):
        ko, po, plo, _ = gpu_segmented(keys, off, pay)
    ek, ep, epl = O.segmented(keys, off, pay)
    assert same_bits(ko, ek) and np.array_equal(po, ep) and np.array_equal(plo, epl)


@pytest.mark.parametrize("m", [511, 1025, 5000])
@pytest.mark.parametrize("wide", [0, 7, 600])
def test_routing_of_many_segments(m, wide):
    """Segments to split in numbers around what the routing workgroups take at
    once: all of them narrow (64 buckets at most), or one in `wide` wider."""
    sizes = np.full(m, 300, dtype=np.uint64) + np.arange(m, dtype=np.uint64) % 700
    if wide:
        sizes[::wide] = 12000
    keys, pay, off = gen.segmented("u32", sizes, ["uniform", "zero", "gaussian"] * (m // 3) + ["uniform"] * (m % 3),
                                   seed=m)
    with R.tuned(cap=256):
        ko, po, plo, _ = gpu_segmented(keys, off, pay)
    ek, ep, epl = O.segmented(keys, off, pay)
    assert same_bits(ko, ek) and np.array_equal(po, ep) and np.array_equal(plo, epl)


@pytest.mark.parametrize("kt,n,values", [("u64", (1 << 20) + 77, 2), ("f32", (1 << 24) + 8191, 300),
                                         ("u64", (1 << 27) - 1, 5), ("u64", 1 << 27, 5), ("u64", (1 << 27) + 8191, 1),
                                         ("u32", (1 << 27) + 1, 2), ("f32", (1 << 27) + 8193, 300)])
def test_equal_splitters_of_all_values(kt, n, values):
    """Few distinct keys, the lowest and the highest bit pattern among them:
    equal splitters, their positions before, inside and after the tiles, below
    and above the size from which the tiles get thresholds of their own."""
    rng = np.random.default_rng(values)
    ut = np.uint64 if kt == "u64" else np.uint32
    top = np.iinfo(ut).max
    v = np.concatenate([np.array([top, 0, top - 1, 1], dtype=ut), rng.integers(0, top, 296, dtype=ut)])[:values]
    x = v[rng.integers(0, values, n, dtype=np.uint32)]
    _check(x.view(np.float32) if kt == "f32" else x, threads=16)


@pytest.mark.parametrize("kt", ["u64", "u32"])
def test_equal_splitters_of_several_segments(kt):
    """The same with a payload and a change of segments between tiles."""
    sizes = np.array([700000, 13000, 90000, 300, 1500000, 14000, 14001], dtype=np.uint64)
    keys, pay, off = gen.segmented(kt, sizes, ["zero", "deterdupl", "uniform", "zero", "deterdupl", "zero", "zero"],
                                   seed=23)
    keys[int(off[0]):int(off[1]):3] = np.iinfo(keys.dtype).max
    ko, po, plo, _ = gpu_segmented(keys, off, pay)
    ek, ep, epl = O.segmented(keys, off, pay)
    assert same_bits(ko, ek) and np.array_equal(po, ep) and np.array_equal(plo, epl)
