"""More than 8 workers of a 16-bit type in large units: the last step of a unit stays in LDS, in the place through which the others
went to the matrix cores.  Units that end anywhere in it, or before it, against the passes over memory and against the units that
are done again from memory."""
import pytest
import torch

from paper_2006_02924_amd import binding as B, workloads as W
from resident_util import steps_and_layers

pytestmark = pytest.mark.gpu
CODE = {torch.bfloat16: B.BF16, torch.float16: B.F16}
STEPS = {9: 5, 10: 5, 11: 5, 12: 5, 13: 4, 14: 4, 15: 4, 16: 4}     # 256 granules of 8 elements each


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("K", sorted(STEPS))
def test_units_that_end_in_the_last_step(K, dtype):
    unit, step = STEPS[K] * 2048, 2048
    tails = [1, 7, 8, 9, 511, 512, 513, 2040, 2047]
    sizes = [unit * 90 + 5] + [unit * 9 - step + t for t in tails] + [unit * 50, unit * 3 - 1, unit + step, 3, unit * 300 + 11]
    offs = W.offsets_from_sizes(sizes)
    steps, units = steps_and_layers(K, offs, CODE[dtype])
    assert steps == STEPS[K] and units.sum() > 512
    print(f"K={K} {dtype}: {units.sum()} units of {steps} steps", flush=True)
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device="cuda", seed=K, scale=W.log_uniform_scales(len(sizes), K, -2.0))
    st = [torch.full((len(sizes), 2), -1.0, dtype=torch.float64, device="cuda") for _ in range(3)]
    got, again, want = (B.adasum_reduce(w.grads, offs, out_dtype=torch.float32, layer_stats=s, **kw)
                        for s, kw in zip(st, ({}, {"resident_wait_us": -1}, {"separate_passes": True})))
    torch.cuda.synchronize()
    assert torch.equal(got, again) and torch.equal(st[0], st[1])
    for l, (a, b) in enumerate(zip(offs, offs[1:])):
        x, y = got[a:b].double(), want[a:b].double()
        # fp32 sums of up to 128 products below the fp64 ones on either side, and one fp32 chain of 8 in the combine
        assert float((x - y).norm()) <= 2e-6 * float(y.norm()), (l, b - a)
    torch.testing.assert_close(st[0], st[2], rtol=2e-6, atol=0)
