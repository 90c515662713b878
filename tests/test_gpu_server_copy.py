"""The sort server's packing copies: requests whose lengths lie around the
pieces a workgroup copies (4096 keys) and the table's chunks (32768), with and
without a permutation, from buffers of any alignment; bit-exact against the
oracle (whole numbers, zero tolerance)."""
import numpy as np
import pytest
import torch

from gen import gen
from oracle import oracle as O
from paper_1606_08766_amd import rsort as R
from tests.gpu_util import banner, dev, host, same_bits

pytestmark = pytest.mark.gpu
LENGTHS = [1, 255, 257, 4095, 4096, 4097, 28673, 32767, 32768, 32769, 36864, 70001]


@pytest.mark.parametrize("kt", ["u64", "u32", "f32"])
@pytest.mark.parametrize("shift", [0, 1])
def test_piece_and_chunk_edges(kt, shift):
    banner("server copies %s shift %d" % (kt, shift))
    xs = [gen.keys(kt, "uniform", n + shift, seed=n)[shift:] for n in LENGTHS]
    ins = [dev(np.concatenate([x[:1]] * shift + [x]))[shift:] for x in xs]
    outs = [(torch.empty_like(dev(np.concatenate([x[:1]] * shift + [x])))[shift:],
             torch.empty(x.size, dtype=torch.uint32, device="cuda") if i % 3 else None) for i, x in enumerate(xs)]
    torch.cuda.synchronize()
    with R.Server(device=0, hbm_budget_bytes=1 << 30, max_inflight=4) as s:
        tickets = [s.submit_tensors(t, o[0], o[1]) for t, o in zip(ins, outs)]
        results = [s.wait(t, 60000) for t in tickets]
    assert all(rc == R.OK for rc, _ in results), [rc for rc, _ in results]
    for x, (ok, op) in zip(xs, outs):
        ek, ep, _ = O.sort(x)
        assert same_bits(ek, host(ok))
        assert op is None or np.array_equal(ep, host(op))
