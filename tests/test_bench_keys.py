"""bench.py joins the library's launch tags to the profiler's kernel names: every
form of one kernel maps to one key, different kernels to different ones, and a
pass with a kernel that was not profiled has no measured traffic."""
import pytest

import bench

A = "(rs::Work, unsigned int, unsigned long const*, unsigned int const*)"
PAIRS = [
    ("(k_local_rank<K, F32, PAY, 512, 12>)", "void rs::k_local_rank<unsigned long, false, false, 512, 12, 4, false>" + A),
    ("(k_local_rank<K, F32, PAY, 512, 8>)", "void rs::k_local_rank<unsigned long, false, false, 512, 8, 6, false>" + A),
    ("(k_local_rank<K, F32, PAY, 1024, 8>)", "void rs::k_local_rank<unsigned long, false, true, 1024, 8, 4, false>" + A),
    ("(k_local_rank<K, F32, PAY, 1024, 8, true>)",
     "void rs::k_local_rank<unsigned long, false, false, 1024, 8, 4, true>" + A),
    ("(k_local_rare<K, F32, PAY, 1024, 8>)", "void rs::k_local_rare<unsigned long, false, true, 1024, 8>" + A),
    ("(k_local_rare<K, F32, PAY, 768, 16>)", "void rs::k_local_rare<unsigned long, false, false, 768, 16>" + A),
    ("(k_split<K, F32, true, PAY, 1024, 8>)",
     "void rs::k_split<unsigned long, false, true, false, 1024, 8, false>" + A),
    ("(k_split<K, F32, true, false, 1024, 8, true>)",
     "void rs::k_split<unsigned long, false, true, false, 1024, 8, true>" + A),
    ("(k_split<K, false, false, PAY, 1024, 8>)",
     "void rs::k_split<unsigned long, false, false, false, 1024, 8, false>" + A),
    ("(k_splitters<K, F32, true, PAY, kSplThreads, kSplItems>)",
     "void rs::k_splitters<unsigned long, false, true, false, 1024, 8>" + A),
    ("(k_splitters<K, false, false, PAY, kSplThreads, kSplItems>)",
     "void rs::k_splitters<unsigned long, false, false, false, 1024, 8>" + A),
    ("k_scan<1024>", "void rs::k_scan<1024>(rs::Work, int)"),
    ("k_route", "rs::k_route(rs::Work, int, rs::LevelEnd)"),
]


@pytest.mark.parametrize("tag,name", PAIRS)
def test_tag_and_profiler_name_share_a_key(tag, name):
    assert bench.kernel_key(tag) == bench.kernel_key(name)


def test_keys_tell_kernels_apart():
    keys = [bench.kernel_key(t) for t, _ in PAIRS]
    assert len(set(keys)) == len(keys)


def test_measured_bytes_need_every_kernel():
    tags = [PAIRS[0][0], PAIRS[1][0]]
    timing = {tags[0]: (4, 1.0), tags[1]: (2, 1.0)}
    t = {"kernels": {bench.kernel_key(tags[0]): {"hbm_bytes_per_launch": 10}}}
    assert bench.measured_bytes(t, timing, tags, 2) is None
    t["kernels"][bench.kernel_key(tags[1])] = {"hbm_bytes_per_launch": 7}
    assert bench.measured_bytes(t, timing, tags, 2) == 27.0
