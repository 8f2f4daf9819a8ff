"""More than 8 workers of a 16-bit type in the resident pass: what the matrix cores sum in fp32 ends at 128 products; everything above
is fp64, however many steps a unit has.  Values whose products a running fp32 sum would drop: 2^24 among a wave's first 128, 1 in
every 128 after them (all exact, also in fp16 and in the products), so the leaves' squared norms come out as whole numbers."""
import pytest
import torch

from paper_2006_02924_amd import binding as B, workloads as W
from resident_util import steps_and_layers

pytestmark = pytest.mark.gpu
CODE = {torch.bfloat16: B.BF16, torch.float16: B.F16}


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("K,steps", [(9, 1), (9, 5), (12, 5), (14, 4), (16, 1), (16, 4)])
def test_no_product_is_dropped(K, steps, dtype):
    unit = steps * 2048
    sizes = [unit * 7] if steps == 1 else [unit * 200] * 4
    offs = W.offsets_from_sizes(sizes)
    found, units = steps_and_layers(K, offs, CODE[dtype])
    assert found == steps, found
    one = torch.zeros(unit, device="cuda")
    one[::128] = 1.0
    one[:2048:512] = 4096.0                   # (a wave's 64 granules of a step are 512 elements)
    g = one.to(dtype).repeat(offs[-1] // unit)
    stats = torch.full((len(sizes), 2), -1.0, dtype=torch.float64, device="cuda")
    B.adasum_reduce([g.clone() for _ in range(K)], offs, layer_stats=stats)
    torch.cuda.synchronize()
    want = [K * int(n) * (4 * 2 ** 24 + unit // 128 - 4) for n in units]
    assert [int(x) for x in stats[:, 1].tolist()] == want
