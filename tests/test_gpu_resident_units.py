"""The resident pass with units of every number of steps a plan can choose, against the definition in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W
from tests.resident_util import LANES, SLOTS, steps_and_layers
from tests.test_gpu_resident import unit_elements, workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {torch.float32: B.F32, torch.bfloat16: B.BF16, torch.float16: B.F16, torch.float64: B.F64}


def pair(a, b):
    d, n1, n2 = torch.dot(a, b), torch.dot(a, a), torch.dot(b, b)
    one = torch.ones_like(d)
    return torch.where(n1 > 0, 1 - d / (2 * n1), one) * a + torch.where(n2 > 0, 1 - d / (2 * n2), one) * b


def tree(grads):
    if len(grads) == 1:
        return grads[0]
    return pair(tree(grads[: len(grads) // 2]), tree(grads[len(grads) // 2:]))


def check(K, dtype, sizes, seed, want_steps):
    w = workload(sizes, K, dtype, seed)
    offs = w.layer_offsets
    steps, units = steps_and_layers(K, offs, CODE[dtype])
    print(f"units: K={K} {dtype} {steps} steps, {units.sum()} units, at most {units.max()} a layer", flush=True)
    assert want_steps is None or steps == want_steps
    wide = torch.float64 if dtype == torch.float64 else torch.float32
    stats = torch.empty(w.n_layers, 2, dtype=torch.float64, device=DEV)
    out = B.adasum_reduce(w.grads, offs, out_dtype=wide, layer_stats=stats)
    flat = torch.empty_like(out)
    B.adasum_reduce(w.grads, offs, flat, out_dtype=wide, noalloc=True)
    assert torch.equal(out, flat)
    tol = 1e-12 if dtype == torch.float64 else 1e-6    # (fp32 lane sums of a few hundred products, one rounding per operand)
    for l, (lo, hi) in enumerate(zip(offs, offs[1:])):
        if hi - lo < 17:                               # (vectors that short may cancel: the definition's own tests have them)
            continue
        want = tree([g[lo:hi].double() for g in w.grads])
        norm = torch.linalg.vector_norm(want)
        assert torch.linalg.vector_norm(out[lo:hi].double() - want) <= tol * norm, l
        assert abs(stats[l, 0] - norm * norm) <= 4 * tol * norm * norm, l


@pytest.mark.parametrize("K,dtype", [(2, torch.bfloat16), (3, torch.float32), (5, torch.float16), (8, torch.float32),
                                     (8, torch.bfloat16), (7, torch.float64), (8, torch.float64), (12, torch.bfloat16),
                                     (16, torch.bfloat16), (12, torch.float32), (16, torch.float32)])
def test_steps_from_few_to_all(K, dtype):
    vec = 16 // torch.empty(0, dtype=dtype).element_size()
    form = 2 if K <= 8 else 3
    most = unit_elements(K, dtype, form) // (LANES * vec)
    slots = SLOTS[form]
    seen = set()
    for n in range(1, most + 1):
        step = LANES * vec
        # 40 layers; half of what the chip holds in units of n steps above what it holds in units of n - 1
        per = int((n - 0.5) * step * slots / 40) + 13
        sizes = [17, per - step + 1, per, 29, step * n, step * n - 1, 33, step * n + 1] + [per + 3 * i - 50 for i in range(36)]
        offs = W.offsets_from_sizes(sizes)
        steps, _ = steps_and_layers(K, offs, CODE[dtype])
        if steps in seen:
            continue
        seen.add(steps)
        check(K, dtype, sizes, 60 + n, None)
    assert most in seen and (most < 3 or len(seen) >= 3), seen


@pytest.mark.parametrize("K,dtype", [(2, torch.bfloat16), (8, torch.float64), (5, torch.float32), (16, torch.bfloat16), (9, torch.float32)])
def test_many_tiny_layers(K, dtype):
    """More units of one step than the chip holds at once: most layers have one, some a few."""
    vec = 16 // torch.empty(0, dtype=dtype).element_size()
    rng = np.random.default_rng(K)
    sizes = [int(s) for s in rng.integers(17, 900, 1500)] + [LANES * vec, LANES * vec * 3 + 5, 15 * LANES * vec - 1, 18, 0, 1]
    rng.shuffle(sizes)
    check(K, dtype, sizes, 80 + K, 1)
