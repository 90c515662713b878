"""Keys that crowd few of the local sort's bins (far outliers, keys spread over
the magnitudes, clusters at the type's ends, one key or two that a part of the
elements share): ranked by place, merge sorted in the same workgroup or handed
to k_local_rare; bit-exact against the oracle (whole numbers, zero
tolerance)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import banner, dev, gpu_segmented, gpu_sort, same_bits

pytestmark = pytest.mark.gpu

FORMS = ["log", "outlier", "halves", "steps", "ends", "spike1", "spike4", "spike15", "spike40"]


def _keys(form, kt, n, rng):
    bits = 64 if kt == "u64" else 32
    r = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    if form == "log":  # as many keys of every magnitude
        k = (r >> np.uint64(64 - bits)) >> rng.integers(0, bits - 1, n, dtype=np.uint64)
    elif form == "outlier":  # small keys, one in 150 anywhere
        k = np.where(rng.random(n) < 1 / 150, r >> np.uint64(64 - bits), r & np.uint64(0xFFF))
    elif form == "halves":  # two clusters far apart
        k = (r & np.uint64(0xFF)) | ((r >> np.uint64(20) & np.uint64(1)) << np.uint64(bits - 1))
    elif form.startswith("spike"):  # a part of the elements share one key, as many another
        k = r >> np.uint64(64 - bits)
        share = rng.random(n)
        k[share < int(form[5:]) / 100] = 0
        k[share > 1 - int(form[5:]) / 100] = 1 << (bits - 3)
    elif form == "steps":  # equal keys, few of every magnitude
        k = np.uint64(1) << rng.integers(0, bits, n, dtype=np.uint64)
    else:  # "ends": the smallest and the largest keys, and those next to them
        k = (r & np.uint64(3)) - (r >> np.uint64(30) & np.uint64(1)) * np.uint64(4)
        k = k & np.uint64((1 << bits) - 1)
    k = k.astype(np.uint64 if bits == 64 else np.uint32)
    return k.view(np.float32) if kt == "f32" else k


@pytest.mark.parametrize("kt", ["u64", "u32", "f32"])
@pytest.mark.parametrize("form", FORMS)
def test_direct_calls(kt, form):
    """One workgroup, at the edges of its shapes and beside them."""
    rng = np.random.default_rng(len(form))
    for n in (2, 100, 255, 256, 257, 289, 1000, 1023, 1024, 1025, 1055, 4065, 4096, 4097, 8161, 8192, 8193, 8255, 12000,
              12287, 12288):
        x = _keys(form, kt, n, rng)
        ek, ep, _ = O.sort(x)
        ko, po = gpu_sort(x)
        assert same_bits(ko, ek) and np.array_equal(po, ep), n


@pytest.mark.parametrize("kt", ["u64", "u32", "f32"])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("payload", [False, True])
def test_segments(kt, form, payload):
    rng = np.random.default_rng(len(form) + 1)
    sizes = [3, 65, 200, 256, 257, 300, 1000, 1024, 1500, 4095, 4096, 4097, 6000, 8191, 8192, 8193, 12288] * 7 + [100_000]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    keys = np.concatenate([_keys(form, kt, n, rng) for n in sizes])
    pay = rng.integers(0, 1 << 32, keys.size, dtype=np.uint64).astype(np.uint32) if payload else None
    ek, ep, ey = O.segmented(keys, off, pay)
    for with_perm in (True, False):
        ko, po, yo, _ = gpu_segmented(keys, off, pay, with_perm=with_perm)
        assert same_bits(ko, ek) and (not with_perm or np.array_equal(po, ep))
        assert not payload or np.array_equal(yo, ey)


def test_crowded_rows_take_little_longer():
    """16384 rows of 256 f32 keys: crowded ones take 1.5 times as long as uniform
    ones (16 times when they were handed over to a launch of large
    workgroups)."""
    rng = np.random.default_rng(5)
    n = 1 << 22
    off = dev(np.arange(0, n + 1, 256, dtype=np.int64))

    def ms(x):
        R.segmented_sort(x, off)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            R.segmented_sort(x, off)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 10

    banner("time of rows of uniform and of crowded keys")
    uniform = ms(dev(rng.random(n, dtype=np.float32)))
    crowded = ms(dev(_keys("log", "f32", n, rng)))
    assert crowded < 5 * uniform, (uniform, crowded)


@pytest.mark.parametrize("rows,length", [(4096, 4096), (2000, 8000)])
def test_shared_keys_take_little_longer(rows, length):
    """Rows of u64 keys, a tenth of which are 0: 3.2 and 4.1 times as long as
    uniform ones (21 and 39 times when every thread ranked its own elements);
    the bound leaves a factor of two."""
    rng = np.random.default_rng(6)
    n = rows * length
    off = dev(np.arange(0, n + 1, length, dtype=np.int64))
    x = rng.integers(0, 1 << 63, n, dtype=np.uint64)

    def ms(t):
        R.segmented_sort(t, off)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            R.segmented_sort(t, off)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 5

    banner("time of rows of uniform keys and of rows with a shared key")
    uniform = ms(dev(x))
    shared = ms(dev(np.where(rng.random(n) < 0.1, np.uint64(0), x)))
    assert shared < 8 * uniform, (uniform, shared)


@pytest.mark.parametrize("kt", ["u64", "u32"])
@pytest.mark.parametrize("n,most", [(12_000, 2.5), (3_145_728, 1.35)])
def test_few_values_rank(kt, n, most):
    """Keys below 16 are ranked and not merge sorted: 1.7 times as long as uniform
    ones where one workgroup sorts them all (4.6 when it merge sorted them), 1.1
    times at 3145728 u64 keys (1.65 when their segments were handed over); the
    bounds lie between."""
    rng = np.random.default_rng(7)
    dt = np.uint64 if kt == "u64" else np.uint32
    x = rng.integers(0, 1 << (63 if kt == "u64" else 31), n, dtype=np.uint64).astype(dt)
    few = rng.integers(0, 16, n).astype(dt)
    ek, ep, _ = O.sort(few)
    ko, po = gpu_sort(few)
    assert same_bits(ko, ek) and np.array_equal(po, ep)

    def ms(t):
        for _ in range(20):
            R.sort(t)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(50):
            R.sort(t)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 50

    banner("time of uniform keys and of keys of few values")
    uniform, shared = ms(dev(x)), ms(dev(few))
    print(n, kt, uniform, shared, flush=True)
    assert shared < most * uniform, (uniform, shared)
