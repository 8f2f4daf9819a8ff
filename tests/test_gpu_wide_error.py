"""The error of an fp32 result against 64 bits: a wide first pass, the default of 16-bit gradients of more than 16
workers, is no further off than the passes of radix 16, and the resident pass no further than the three kernels."""
import pytest
import torch

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def exact(grads):
    """The definition over one layer, in 64 bits."""
    if len(grads) == 1:
        return grads[0].double()
    a, b = exact(grads[: len(grads) // 2]), exact(grads[len(grads) // 2:])
    d = torch.dot(a, b)
    return (1 - d / (2 * torch.dot(a, a))) * a + (1 - d / (2 * torch.dot(b, b))) * b


@pytest.mark.parametrize("K", [17, 24, 40, 64])
def test_no_further_off_than_radix_16(K):
    """Over 5 million independent elements the norm of the error is the sum of its sources' variances, so the two
    figures repeat to a per cent; a tenth is left for it."""
    print(f"error of the wide pass K={K}", flush=True)
    w = W.correlated_gaussian([5_000_003], K, dtype=torch.bfloat16, device=DEV, seed=4)
    ref = exact(w.grads)
    wide, narrow = (torch.linalg.vector_norm(B.adasum_reduce(w.grads, w.layer_offsets, out_dtype=torch.float32, radix=r).double() - ref)
                    for r in (0, 16))
    assert wide <= 1.1 * narrow, (float(wide), float(narrow))


@pytest.mark.parametrize("K,dtype", [(2, torch.bfloat16), (8, torch.bfloat16), (9, torch.bfloat16), (12, torch.bfloat16), (16, torch.bfloat16),
                                     (8, torch.float32), (16, torch.float32)])
def test_the_resident_pass_no_further_off_than_three_kernels(K, dtype):
    """As above; a twentieth is left."""
    print(f"error of the resident pass K={K} {dtype}", flush=True)
    sizes = [1_250_001, 1_249_999, 1_250_003, 1_250_000]
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device=DEV, seed=4)
    code = {torch.float32: B.F32, torch.bfloat16: B.BF16}[dtype]
    need, without = (B.adasum_workspace_bytes(K, w.layer_offsets, code, out_dtype_code=B.F32, separate_passes=s) for s in (False, True))
    assert need > without                      # (taken as a resident pass)
    ref = torch.cat([exact([g[lo:hi] for g in w.grads]) for lo, hi in zip(w.layer_offsets, w.layer_offsets[1:])])
    one, three = (torch.linalg.vector_norm(B.adasum_reduce(w.grads, w.layer_offsets, out_dtype=torch.float32, separate_passes=s).double() - ref)
                  for s in (False, True))
    assert one <= 1.05 * three, (float(one), float(three))
