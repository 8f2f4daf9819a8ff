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


@pytest.mark.parametrize("K,sizes,radix", [
    # few layers of some million elements: [16, 4] is faster than [32, 2] up to 48 workers
    (33, [1_000_000], 16), (48, [700_000], 16), (48, [699_999], 32), (33, [2_999_999], 16), (33, [3_000_000], 32),
    (49, [1_000_000], 32), (32, [1_000_000], 32), (40, [60_000] * 20, 16), (40, [60_000] * 19 + [59_999], 32),
    # beyond 64 workers passes of 64 pay later
    (65, [7_999_999], 32), (65, [8_000_000], 64), (64, [7_999_999], 64)])
def test_the_default_where_radices_change_places(K, sizes, radix):
    """The default is the named schedule bit for bit, and not the other ones."""
    print(f"default radix K={K} {len(sizes)} layers of {sizes[0]}", flush=True)
    offs = W.offsets_from_sizes(sizes)
    gen = torch.Generator(device=DEV).manual_seed(K)
    base = torch.randn(offs[-1], device=DEV, generator=gen)
    grads = [(base + 0.7 * torch.randn(offs[-1], device=DEV, generator=gen)).to(torch.bfloat16) for _ in range(K)]
    got = B.adasum_reduce(grads, offs, out_dtype=torch.float32)
    same = {r: torch.equal(got, B.adasum_reduce(grads, offs, out_dtype=torch.float32, radix=r)) for r in (16, 32, 64)}
    assert same[radix] and not all(same.values()), same
    if K <= 32:
        assert same[64]        # (64 is 32 up to 32 workers)
    else:
        assert sum(same.values()) == 1, same


def test_shapes_with_a_small_workspace_take_one_place_each_in_the_plan_cache():
    """40 shapes whose workspaces have no room for the resident pass: 40 plans of the 64 that are kept, so the second
    round through them makes none.  (Making one takes a dozen device allocations and copies, some hundred us.)"""
    import time
    B.shutdown()
    shapes = [(W.offsets_from_sizes([1000 + i, 70_000 + 3 * i, 33]), i) for i in range(40)]
    grads = [torch.randn(90_000, device=DEV) for _ in range(8)]
    ws = []
    for offs, _ in shapes:
        small = B.adasum_workspace_bytes(8, offs, B.F32, separate_passes=True)
        assert small < B.adasum_workspace_bytes(8, offs, B.F32)
        ws.append(torch.empty(small, dtype=torch.uint8, device=DEV))
    took = []
    for turn in range(4):
        if turn == 1:                      # (the first round loaded the kernels)
            B.shutdown()
        torch.cuda.synchronize()
        t = time.perf_counter()
        for (offs, i), w in zip(shapes, ws):
            n = offs[-1]
            out = torch.empty(n, device=DEV)
            B.adasum_reduce([g[:n] for g in grads], offs, out, workspace=w)
        torch.cuda.synchronize()
        took.append(time.perf_counter() - t)
    print(f"rounds: {[round(1e3 * x, 2) for x in took]} ms", flush=True)
    assert min(took[2:]) < 0.5 * took[1]
    # with room for it the resident pass is taken, beside the lean plan of the same shape
    offs = shapes[0][0]
    roomy = torch.empty(B.adasum_workspace_bytes(8, offs, B.F32), dtype=torch.uint8, device=DEV)
    views = [g[: offs[-1]] for g in grads]
    for _ in range(2):
        assert torch.equal(B.adasum_reduce(views, offs, workspace=roomy), B.adasum_reduce(views, offs))
        a = B.adasum_reduce(views, offs, workspace=ws[0])
        b = B.adasum_reduce(views, offs, separate_passes=True)
        assert torch.equal(a, b)
