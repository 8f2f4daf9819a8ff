"""The resident pass (a single pass that keeps what it has read): sizes around its units, every form it takes, the
number of units at which the exchange changes, layers just too large for it, and waits that end unanswered."""
import numpy as np
import pytest
import torch

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W
from tests.gpu_util import assert_parity, oracle_after_optimizer, oracle_reduce

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LANES = 256                                   # granules of a step


def unit_elements(K, dtype, form, delta=False):
    """Elements of a full unit (adasum_host.h: resident_steps)."""
    vec = 16 // torch.empty(0, dtype=dtype).element_size()
    rows = K + (1 if delta else 0)
    if form == 1:
        return LANES * vec
    if K > 8:
        rows = (K + 1) // 2 * 2
    matrix = K > 8 and vec == 8
    short = rows == 8 or (rows >= 7 and dtype == torch.float64)
    registers = {2: 16 if short else 21 if rows == 3 else 24, 3: 48 if matrix else 32 if dtype == torch.float64 or K > 8 else 40}[form]
    steps = max(1, min(16, registers // rows)) + (0 if matrix else min(8, {2: 12, 3: 18}[form] // rows))
    return LANES * vec * steps


def workload(sizes, K, dtype, seed):
    wide = torch.float32 if dtype == torch.float64 else dtype
    scale = W.log_uniform_scales(len(sizes), seed, -2.0, 0.0) if dtype == torch.float16 else None
    w = W.correlated_gaussian(sizes, K, dtype=wide, device=DEV, seed=seed, scale=scale)
    if dtype == torch.float64:
        w.grads, w.dtype = [g.double() for g in w.grads], dtype
    return w


def edges(u, vec):
    """Layers around a unit's capacity, and around the number of units where every workgroup stops reading all sums."""
    return [u, 1, vec - 1 if vec > 2 else 3, u - 1, u + 1, 17, 2 * u + vec, 0, 16 * u - 40, 16 * u + 1, 33, 17 * u + 5, vec]


CASES = [(K, dtype, form) for form in (1, 2, 3) for K, dtype in (
    (2, torch.bfloat16), (3, torch.float32), (4, torch.float64), (5, torch.float16), (6, torch.bfloat16),
    (7, torch.float32), (8, torch.float32), (8, torch.bfloat16), (8, torch.float64))] + [
    # more than 8 operands have no form 2; 16-bit ones on the matrix cores, odd counts filled up
    (K, dtype, form) for form in (1, 3) for K, dtype in (
        (9, torch.bfloat16), (12, torch.bfloat16), (14, torch.float16), (16, torch.bfloat16), (11, torch.float32),
        (16, torch.float32))]


@pytest.mark.parametrize("K,dtype,form", CASES)
def test_unit_edges_against_the_oracle(K, dtype, form):
    vec = 16 // torch.empty(0, dtype=dtype).element_size()
    u = unit_elements(K, dtype, form)
    sizes = edges(u, vec)
    if form == 2:      # more units of one step than the chip holds at once
        sizes.append(max(0, 769 * unit_elements(K, dtype, 1) - sum(sizes)) + 7)
    elif form == 3 and K <= 8:    # a layer of more than half the units of form 2
        sizes.append(385 * unit_elements(K, dtype, 2) + 3)
    elif form == 3:
        sizes.append(max(0, 769 * unit_elements(K, dtype, 1) - sum(sizes)) + 7)
    print(f"resident K={K} {dtype} form {form}: unit {u}, N={sum(sizes)}", flush=True)
    w = workload(sizes, K, dtype, 40 + K)
    wide = torch.float64 if dtype == torch.float64 else torch.float32
    stats = torch.full((w.n_layers, 2), -1.0, dtype=torch.float64, device=DEV)
    out = B.adasum_reduce(w.grads, w.layer_offsets, out_dtype=wide, layer_stats=stats)
    again = B.adasum_reduce(w.grads, w.layer_offsets, out_dtype=wide)
    ref = oracle_reduce(w.grads, w.layer_offsets)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    assert_parity(out, ref, w.layer_offsets, what=f"form {form}")
    got = stats.cpu().numpy()
    offs = w.layer_offsets
    leaves = [g.double() for g in w.grads]
    for l in range(w.n_layers):
        lo, hi = offs[l], offs[l + 1]
        # fp32 lane sums: a run of at most a few hundred products per lane
        assert np.isclose(got[l, 1], sum(float((g[lo:hi] * g[lo:hi]).sum()) for g in leaves), rtol=1e-6, atol=0)
        if hi > lo and not np.isnan(ref[lo:hi]).any():
            assert np.isclose(got[l, 0], float(np.dot(ref[lo:hi], ref[lo:hi])), rtol=4e-6, atol=0), l
    # the same bits from the entry point without allocation and in a workspace of the caller's
    flat = torch.empty_like(out)
    B.adasum_reduce(w.grads, w.layer_offsets, flat, out_dtype=wide, noalloc=True)
    code = {torch.float32: B.F32, torch.bfloat16: B.BF16, torch.float16: B.F16, torch.float64: B.F64}
    n = B.adasum_workspace_bytes(K, offs, code[dtype], out_dtype_code=code[wide])
    ws = torch.full((n,), 0x5a, dtype=torch.uint8, device=DEV)
    own = B.adasum_reduce(w.grads, offs, out_dtype=wide, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(out, flat) and torch.equal(out, own)


@pytest.mark.parametrize("K,dtype", [(8, torch.float32), (4, torch.bfloat16)])
def test_a_layer_just_too_large_takes_the_other_passes(K, dtype):
    u = unit_elements(K, dtype, 3)
    sizes = [700, 500 * u, 3 * u + 1]      # 500 units: the largest that is kept
    for extra in (0, 1):
        sizes[1] = 499 * u + extra + (u - 700 % u)     # exactly 500 cells, or one more
        w = workload(sizes, K, dtype, 9)
        out = B.adasum_reduce(w.grads, w.layer_offsets, out_dtype=torch.float32)
        ref = oracle_reduce(w.grads, w.layer_offsets)
        assert_parity(out, ref, w.layer_offsets, what=f"{sizes[1]} elements")


@pytest.mark.parametrize("K,dtype", [(8, torch.bfloat16), (3, torch.float32)])
def test_after_optimizer_form(K, dtype):
    u = unit_elements(K, dtype, 2, delta=True)
    sizes = [5, u + 1, 3 * u - 9, 769 * unit_elements(K, dtype, 1)]
    w = W.after_local_step(sizes, K, dtype=dtype, device=DEV, seed=12, step=0.25)
    start = w.meta["start"]
    ref = oracle_after_optimizer(start, w.grads, w.layer_offsets, range(len(sizes)))
    out = B.adasum_reduce(w.grads, w.layer_offsets, delta_start=start)
    inplace = start.clone()
    B.adasum_reduce(w.grads, w.layer_offsets, inplace, delta_start=inplace)
    torch.cuda.synchronize()
    assert_parity(out, ref, w.layer_offsets, what="after the optimizer")
    assert torch.equal(out, inplace)


def test_two_streams_that_each_want_the_whole_chip():
    """Two plans at once, each with layers of more than half the chip: neither can have all of a layer's workgroups
    running at times, waits end unanswered, and the second launch does the rest.  The results are the same bits."""
    K, sizes = 8, [1 << 21, 1000, 1 << 21, (1 << 21) - 3]
    loads = [workload(sizes, K, torch.float32, 70 + i) for i in range(2)]
    plans = [B.Plan(K, w.layer_offsets, torch.float32) for w in loads]
    alone = [p.execute(w.grads) for p, w in zip(plans, loads)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in loads]
    outs = [torch.empty_like(a) for a in alone]
    for rep in range(3):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(4):
            for p, w, o, s in zip(plans, loads, outs, streams):
                p.execute(w.grads, o, stream=s)
        torch.cuda.synchronize()
        for a, o in zip(alone, outs):
            assert torch.equal(a, o), rep


def test_captured_by_the_caller_and_replayed():
    """The tag that tells one call's sums from another's lives on the device: replays of one capture have their own."""
    K, sizes = 4, [3000, 17, 900000, 1]
    w = workload(sizes, K, torch.float32, 5)
    plan = B.Plan(K, w.layer_offsets, torch.float32)
    out, eager = torch.empty(w.N, device=DEV), torch.empty(w.N, device=DEV)
    plan.execute(w.grads, eager)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(w.grads, out)
    for rep in range(4):
        for i, t in enumerate(w.grads):
            t.mul_(1.0 + 0.5 * ((i + rep) % 3)).add_(0.01 * rep)
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        plan.execute(w.grads, eager)
        torch.cuda.synchronize()
        assert torch.equal(out, eager), rep
