"""Segment offsets that are not a partition of the input: the call sets the
workspace status and touches nothing beyond its workspace and outputs, also
where the segments overlap and together are many times as long as the input."""
import numpy as np
import pytest
import torch

from gen import gen
from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import banner, dev, gpu_segmented, same_bits

pytestmark = pytest.mark.gpu

N = (1 << 20) + 5
GUARD = 1 << 16


def _offsets(form):
    if form == "overlap_split":  # 40 segments of all keys, each of which would be split
        return [0, N] * 40
    if form == "overlap_small":  # 3000 segments of 5000 keys on the same keys
        return [0] + [100, 5100] * 3000 + [N]
    if form == "overlap_across":  # a bad entry in another workgroup's share than the segments
        return [0] + [N] * 5000 + [7, N]
    if form == "late_end":
        return [0, 5, 200000, N + 1]
    if form == "late_start":
        return [3, 5, 200000, N]
    return [0, 5, 200000, N - 1]  # "early_end"


@pytest.mark.parametrize("form", ["overlap_split", "overlap_small", "overlap_across", "late_end", "late_start",
                                  "early_end"])
@pytest.mark.parametrize("payload", [False, True])
def test_bad_offsets_set_the_status_only(form, payload):
    off = np.array(_offsets(form), dtype=np.int64)
    x = gen.keys("u64", "uniform", N, seed=2)
    pay = gen.payload(N) if payload else None
    need = R.segmented_workspace_bytes(R.U64, N, off.size - 1, payload)
    ws = torch.full((need + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    ko = torch.full((8 * N + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    po = torch.full((4 * N + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    yo = torch.full((4 * N + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    banner("bad offsets %s payload=%s" % (form, payload))
    R.segmented_sort(dev(x), dev(off), dev(pay) if payload else None, workspace=ws[:need],
                     out=(ko[:8 * N].view(torch.uint64), po[:4 * N].view(torch.uint32),
                          yo[:4 * N].view(torch.uint32) if payload else None))
    assert R.workspace_status(ws) == R.EINVAL
    for t, size in ((ws, need), (ko, 8 * N), (po, 4 * N), (yo, 4 * N)):
        assert bool((t[size:] == 0x5A).all())
    # the same workspace sizes serve a good call afterwards
    good = np.array([0, 300000, 300100, N], dtype=np.uint64)
    gk, gp, gy, _ = gpu_segmented(x, good, pay)
    ek, ep, ey = O.segmented(x, good, pay)
    assert same_bits(gk, ek) and np.array_equal(gp, ep) and (not payload or np.array_equal(gy, ey))
