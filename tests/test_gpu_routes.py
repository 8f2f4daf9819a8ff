"""Calls that another entry point, workspace or device load sends another way: the result is the same."""
import pytest
import torch

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("K,dtype,sizes", [(16, torch.bfloat16, [3_000] * 8_000), (8, torch.float32, [129] * 40_000)])
def test_noalloc_gives_the_same_bits_where_the_resident_pass_does_not_fit_its_scratch(K, dtype, sizes):
    print(f"noalloc K={K} {dtype} {len(sizes)} layers", flush=True)
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device=DEV, seed=8)
    out = torch.full((w.N,), float("nan"), dtype=dtype, device=DEV)
    B.adasum_reduce(w.grads, w.layer_offsets, out, noalloc=True)
    assert torch.equal(out, B.adasum_reduce(w.grads, w.layer_offsets))
    plan = B.Plan(K, w.layer_offsets, dtype)
    assert torch.equal(out, plan.execute(w.grads))
