"""The default radix of 16-bit gradients around the sizes where it changes: the default is the named schedule bit for
bit, and takes magnitudes as large as the other schedules do."""
import numpy as np
import pytest
import torch

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W
from tests.gpu_util import oracle_reduce

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("K,N,radix", [(16, 70_001, 16), (17, 70_001, 32), (32, 70_001, 32), (33, 3_999_999, 32),
                                       (33, 4_000_000, 64), (32, 4_000_000, 32), (65, 70_001, 32)])
def test_default_is_the_named_schedule(K, N, radix, dtype):
    print(f"default radix K={K} N={N} {dtype}", flush=True)
    sizes = [1, 17, 5_003, 0, 33, N - 5_054]
    scale = W.log_uniform_scales(len(sizes), 3, -2.0, 0.0) if dtype == torch.float16 else None
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device=DEV, seed=3, scale=scale)
    got = B.adasum_reduce(w.grads, w.layer_offsets)
    assert torch.equal(got, B.adasum_reduce(w.grads, w.layer_offsets, radix=radix))
    if N < 100_000:
        out = torch.empty_like(got)
        B.adasum_reduce(w.grads, w.layer_offsets, out, noalloc=True)
        assert torch.equal(got, out)


@pytest.mark.parametrize("K,dtype,code,enough", [(16, torch.float32, B.F32, 24_320), (8, torch.float64, B.F64, 9_216),
                                                 (33, torch.bfloat16, B.BF16, 1_318_912)])
def test_a_workspace_without_room_for_the_faster_passes(K, dtype, code, enough):
    """`enough` is what the passes without the resident one and without a wide default take: refused below it, and
    from it on the result of those passes (within rounding: separate passes sum the same products in other orders)."""
    print(f"lean workspace K={K} {dtype}", flush=True)
    offs = W.offsets_from_sizes([1, 17, 5_003, 33, 70_001])
    assert B.adasum_workspace_bytes(K, offs, code) > enough
    wide = torch.float32 if dtype == torch.float64 else dtype
    w = W.correlated_gaussian([1, 17, 5_003, 33, 70_001], K, dtype=wide, device=DEV, seed=9)
    grads = [g.to(dtype) for g in w.grads]
    out_dtype = torch.float64 if dtype == torch.float64 else torch.float32
    ws = torch.empty(enough, dtype=torch.uint8, device=DEV)
    got = B.adasum_reduce(grads, offs, out_dtype=out_dtype, workspace=ws)
    ref = oracle_reduce(grads, offs)
    own = B.adasum_reduce(grads, offs, out_dtype=out_dtype)
    # both are within half an fp32 epsilon times a small factor of the exact result per layer
    tol = 1e-13 if dtype == torch.float64 else 2e-6
    for lo, hi in zip(offs[:-1], offs[1:]):
        assert torch.linalg.vector_norm((got - own)[lo:hi].double()) <= tol * torch.linalg.vector_norm(own[lo:hi].double())
        if not np.isnan(ref[lo:hi]).any():               # (a layer whose result is ill-posed has no reference)
            d = got[lo:hi].cpu().double().numpy() - ref[lo:hi]
            assert np.linalg.norm(d) <= tol * np.linalg.norm(ref[lo:hi])
    plan = B.Plan(K, offs, dtype, out_dtype=out_dtype, workspace=ws)
    out = torch.empty_like(got)
    plan.execute(grads, out)
    assert torch.equal(out, got)
    with pytest.raises(Exception):
        B.adasum_reduce(grads, offs, out_dtype=out_dtype, workspace=ws[: enough - 256])


@pytest.mark.parametrize("K", [24, 40])
def test_magnitudes_of_the_other_schedules(K):
    """Layers of rms 7e16, scaled by a power of two: every sum scales exactly, so the result does."""
    print(f"default radix, large values K={K}", flush=True)
    w = W.correlated_gaussian([4_111, 300_000], K, dtype=torch.bfloat16, device=DEV, seed=5, scale=np.ones(2))
    big = 2.0 ** 56                                              # 7.2e16; the generator's rows have rms about 1
    small = B.adasum_reduce(w.grads, w.layer_offsets, out_dtype=torch.float32)
    large = B.adasum_reduce([g * big for g in w.grads], w.layer_offsets, out_dtype=torch.float32)
    assert torch.isfinite(large).all() and torch.equal(large, small * big)
