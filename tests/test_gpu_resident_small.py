"""Layers of at most 16 elements in a reduction that is taken as a resident pass: by the definition, with the bits that the passes
over memory give them, wherever a unit's boundary cuts them; and the larger layers beside them, which they must leave alone."""
import math

import pytest
import torch

from paper_2006_02924_amd import binding as B, workloads as W
from resident_util import LANES, steps_and_layers

pytestmark = pytest.mark.gpu
DEV = "cuda"
CODE = {torch.float32: B.F32, torch.bfloat16: B.BF16, torch.float16: B.F16, torch.float64: B.F64}
VEC = {torch.float32: 4, torch.bfloat16: 8, torch.float16: 8, torch.float64: 2}
BIG = [[30_000], [400_000] * 16]     # small units in one launch; larger ones and a second launch
SMALL = list(range(1, 17)) + [1, 1, 16, 3]


def table(K, dtype, big, **kw):
    """Small layers among larger ones, one of them across a boundary between two units."""
    sizes = [5000] + SMALL[:9] + big + SMALL[9:]
    for _ in range(4):
        steps, _ = steps_and_layers(K, W.offsets_from_sizes(sizes + [12, 700]), CODE[dtype], **kw)
        cap = steps * LANES * VEC[dtype]
        sizes[-1 - len(SMALL[9:])] += -(sum(sizes) + 5) % cap          # (the layer after these starts 5 elements before a boundary)
        full = sizes + [12, 700]
        if steps_and_layers(K, W.offsets_from_sizes(full), CODE[dtype], **kw)[0] == steps and (sum(sizes) + 5) % cap == 0:
            break
    else:
        raise AssertionError("no table found")
    _, per_layer = steps_and_layers(K, W.offsets_from_sizes(full), CODE[dtype], **kw)
    assert per_layer[-2] == 2
    return full, steps


def assert_larger_layers_close(got, want, offs, K, dtype):
    """Two ways of summing: runs of up to 128 products in the lanes' type at each of the tree's levels and a chain of K in the combine,
    and a rounding of the result on either side.  Element by element too: a single wrong one hardly shows in a layer's norm."""
    lane = 2.0 ** (-53 if dtype == torch.float64 else -24)
    sums = (128 * math.ceil(math.log2(K)) + K) * lane if dtype != torch.float64 else 1e4 * lane    # (fp64: all sums, 4e5 terms in some 1e3 in a row)
    ulp = {torch.bfloat16: 2.0 ** -7, torch.float16: 2.0 ** -10}.get(dtype, 0.0)
    for l, (a, b) in enumerate(zip(offs, offs[1:])):
        if b - a > 16:
            x, y = got[a:b].double(), want[a:b].double()
            assert float((x - y).norm()) <= (sums + ulp / 2) * float(y.norm()), (l, b - a)
            atol = 6 * K * sums * float(y.norm()) / math.sqrt(b - a)      # (K weights off by `sums`, elements of six standard deviations)
            assert bool(((x - y).abs() <= ulp * y.abs() + atol).all()), (l, b - a)


CASES = [(2, torch.bfloat16), (3, torch.float16), (5, torch.float32), (8, torch.float32), (8, torch.float64), (7, torch.bfloat16),
         (9, torch.bfloat16), (12, torch.float32), (16, torch.bfloat16)]


@pytest.mark.parametrize("order", ["tree", "linear"])
@pytest.mark.parametrize("big", BIG)
@pytest.mark.parametrize("K,dtype", CASES)
def test_same_bits_as_the_passes_over_memory(K, dtype, big, order):
    if order == "linear" and K not in (2, 8, 16):
        pytest.skip("more than one pass in this order")
    kw = {"order": B.ORDER_LINEAR if order == "linear" else B.ORDER_TREE}
    sizes, steps = table(K, dtype, big, **kw)
    print(f"K={K} {dtype} {order}: units of {steps} steps", flush=True)
    w = W.correlated_gaussian(sizes, K, dtype=dtype, device=DEV, seed=K)
    stats = [torch.full((w.n_layers, 2), -1.0, dtype=torch.float64, device=DEV) for _ in range(2)]
    got = B.adasum_reduce(w.grads, w.layer_offsets, layer_stats=stats[0], **kw)
    want = B.adasum_reduce(w.grads, w.layer_offsets, layer_stats=stats[1], separate_passes=True, **kw)
    plain = B.adasum_reduce(w.grads, w.layer_offsets, **kw)
    again = torch.empty_like(plain)
    B.adasum_reduce(w.grads, w.layer_offsets, again, noalloc=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(got, plain) and torch.equal(got, again)
    assert_larger_layers_close(got, want, w.layer_offsets, K, dtype)
    for l, n in enumerate(sizes):
        if n <= 16:
            a, b = w.layer_offsets[l], w.layer_offsets[l + 1]
            assert torch.equal(got[a:b], want[a:b]), (l, n)
            # a sum of at most 16 squares in another order
            torch.testing.assert_close(stats[0][l], stats[1][l], rtol=16 * 2.3e-16, atol=0)


@pytest.mark.parametrize("big", BIG)
@pytest.mark.parametrize("K,dtype", [(4, torch.float32), (8, torch.bfloat16), (3, torch.float64)])
def test_after_optimizer_form_in_place(K, dtype, big):
    sizes, _ = table(K, dtype, big, delta=True)
    w = W.after_local_step(sizes, K, dtype=dtype, device=DEV, seed=3, step=0.25)
    start = w.meta["start"]
    want = B.adasum_reduce(w.grads, w.layer_offsets, delta_start=start, separate_passes=True)
    beside = B.adasum_reduce(w.grads, w.layer_offsets, delta_start=start)
    got = start.clone()
    B.adasum_reduce(w.grads, w.layer_offsets, got, delta_start=got)
    torch.cuda.synchronize()
    assert torch.equal(got, beside)
    assert_larger_layers_close(got, want, w.layer_offsets, K, dtype)
    for l, n in enumerate(sizes):
        if n <= 16:
            a, b = w.layer_offsets[l], w.layer_offsets[l + 1]
            assert torch.equal(got[a:b], want[a:b]), (l, n)
