"""Small reductions in one launch each, several at once on streams of their own: their last workgroups wait for the units of their own
launch while the others' hold parts of the chip.  The same bits as alone."""
import pytest
import torch

from paper_2006_02924_amd import binding as B, workloads as W
from resident_util import SLOTS, steps_and_layers

pytestmark = pytest.mark.gpu
CODE = {torch.float32: B.F32, torch.bfloat16: B.BF16, torch.float16: B.F16, torch.float64: B.F64}
LANES = {torch.float32: 1024, torch.bfloat16: 2048, torch.float16: 2048, torch.float64: 512}


@pytest.mark.parametrize("wait", [0, 1, -1])
@pytest.mark.parametrize("shape", [(2, torch.bfloat16), (4, torch.float32), (8, torch.float16), (3, torch.float64)])
def test_side_by_side(shape, wait):
    K, dtype = shape
    n = LANES[dtype]
    streams, plans, outs, wants, loads = [], [], [], [], []
    for i in range(6):
        sizes = [[n * 340 - 9] * 2, [n * 3] * 150 + [7], [n - 1] * 350, [1000, 4096, 65536], [n * 90] * 7 + [1] * 5, [n * 40 + i] * 16][i]
        w = W.correlated_gaussian(sizes, K, dtype=dtype, device="cuda", seed=i)
        steps, units = steps_and_layers(K, w.layer_offsets, CODE[dtype])
        assert steps == 1 and units.sum() <= SLOTS[1]
        wants.append(B.adasum_reduce(w.grads, w.layer_offsets))
        outs.append(torch.empty_like(wants[-1]))
        plans.append(B.Plan(K, w.layer_offsets, dtype, resident_wait_us=wait))
        loads.append(w.grads)
        streams.append(torch.cuda.Stream())
    torch.cuda.synchronize()
    for rep in range(30):
        for s, p, o, g in zip(streams, plans, outs, loads):
            with torch.cuda.stream(s):
                o.fill_(float("nan"))
                p.execute(g, o)
        if rep % 10 == 9:
            torch.cuda.synchronize()
            for i, (o, want) in enumerate(zip(outs, wants)):
                assert torch.equal(o, want), (rep, i)
    print(f"K={K} {dtype} wait {wait}: six streams, 30 calls each", flush=True)
