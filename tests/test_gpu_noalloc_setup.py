"""The entry point that allocates nothing builds the resident pass's tables on the device: the same bits as with tables from the host,
around the number of layers that fit one launch's arguments, with empty and small layers, more units than the chip holds at once,
and memory that an earlier call left behind."""
import random

import pytest
import torch

from paper_2006_02924_amd import binding as B, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,most", [(1, 900_000), (2, 17), (64, 20_000), (255, 3_000), (257, 3_000), (382, 40_000), (383, 40_000),
                                         (384, 40_000), (600, 9_000)])
@pytest.mark.parametrize("K,dtype", [(2, torch.bfloat16), (6, torch.float16), (8, torch.float32), (4, torch.float64)])
def test_same_bits_as_tables_from_the_host(layers, most, K, dtype):
    r = random.Random(layers)
    sizes = [r.choice([0, 1, 16, r.randint(1, most), r.randint(most // 2, most)]) for _ in range(layers)] if layers > 2 else [most] * layers
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device="cuda", seed=layers)
    st = [torch.full((layers, 2), -1.0, dtype=torch.float64, device="cuda") for _ in range(2)]
    want = B.adasum_reduce(w.grads, w.layer_offsets, layer_stats=st[0])
    for _ in range(2):
        got = torch.full_like(want, float("nan"))
        B.adasum_reduce(w.grads, w.layer_offsets, got, noalloc=True, layer_stats=st[1])
        torch.cuda.synchronize()
        assert torch.equal(want, got) and torch.equal(st[0], st[1])
