"""An error that the calling thread left behind before a call -- of another HIP call than the library's -- does not keep the second
launch of a resident pass from following the first: the call is whole, and so is the one after it."""
import pytest
import torch

from paper_2006_02924_amd import binding as B, workloads as W
from resident_util import steps_and_layers

pytestmark = pytest.mark.gpu
INVALID_DEVICE = 101


@pytest.mark.parametrize("K,dtype,sizes", [(2, torch.bfloat16, [20_000_000, 5_000_000, 9]), (8, torch.float32, [3_000_000, 3_000_000, 100]),
                                           (16, torch.bfloat16, [900_000, 900_000, 2_200_000])])
def test_both_launches_of_a_held_plan(K, dtype, sizes):
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device="cuda", seed=K)
    assert steps_and_layers(K, w.layer_offsets, {torch.float32: B.F32, torch.bfloat16: B.BF16}[dtype])[0] > 1
    held, fresh = (B.Plan(K, w.layer_offsets, dtype) for _ in range(2))
    got, want = (torch.empty(w.layer_offsets[-1], dtype=dtype, device="cuda") for _ in range(2))
    lib = B.load()
    held.execute(w.grads, got)
    for rep in range(2):
        for i, t in enumerate(w.grads):
            t.mul_(1.0 + 0.25 * (i + rep))
        torch.cuda.synchronize()
        assert lib.hipSetDevice(1 << 20) == INVALID_DEVICE      # (the runtime refuses it and remembers that)
        try:
            held.execute(w.grads, got)
        finally:
            lib.hipGetLastError()
        fresh.execute(w.grads, want)
        torch.cuda.synchronize()
        assert torch.equal(got, want), rep
