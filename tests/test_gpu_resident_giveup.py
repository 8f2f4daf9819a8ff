"""Units of the resident pass that give up waiting for their layer's others are done by its second launch, with the same
bits.  The wait is set from the host: none at all sends every unit of a layer of several through that launch."""
import pytest
import torch

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W
from tests.resident_util import steps_and_layers
from tests.test_gpu_resident import unit_elements, workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {torch.float32: B.F32, torch.bfloat16: B.BF16, torch.float16: B.F16, torch.float64: B.F64}


class Shape:
    """Layers of one unit, two, the most that exchange directly, more; ragged ends; in forms 2 and 3 more
    of them than the chip holds at once, so that the units are as large as the form has them."""

    def __init__(self, K, dtype, form, delta=False):
        self.K, self.dtype, self.delta = K, dtype, delta
        vec = 16 // torch.empty(0, dtype=dtype).element_size()
        u = unit_elements(K, dtype, form, delta)
        self.sizes = [7, u - 7, u + vec + 3, 0, 16 * u - vec, 17 * u + 5, 33, 70 * u]
        if form == 2:
            self.sizes += [300 * u + 1, 300 * u]
        elif form == 3 and K <= 8:    # a layer of more than half the units of form 2
            self.sizes += [385 * unit_elements(K, dtype, 2, delta) + 3, 200 * u]
        elif form == 3:
            self.sizes += [200 * u + 1, 250 * u]
        self.offs = W.offsets_from_sizes(self.sizes)
        steps, per_layer = steps_and_layers(K, self.offs, CODE[dtype], delta=delta)
        self.units, self.waiting = int(per_layer.sum()), int(per_layer[per_layer > 1].sum())
        self.base = B.adasum_workspace_bytes(K, self.offs, CODE[dtype], delta=delta, separate_passes=True)
        need = B.adasum_workspace_bytes(K, self.offs, CODE[dtype], delta=delta)
        self.workspace = torch.full((need,), 0x5a, dtype=torch.uint8, device=DEV)
        print(f"give up: K={K} {dtype} form {form}, {steps} steps, {self.units} units, {self.waiting} in layers of several", flush=True)

    def redone(self):
        """Units that the second launch did in the call before (the state begins where the other passes' sections end:
        a counter of calls, then a word per unit)."""
        torch.cuda.synchronize()
        words = self.workspace[self.base:][: 4 * (1 + self.units)].view(torch.int32)
        assert int(words[0]) == 1 and int(words[1:].min()) >= 0 and int((words[1:] == 1).sum()) == 0
        return int((words[1:] == 2).sum())


CASES = [(K, dtype, form) for form in (1, 2, 3) for K, dtype in (
    (2, torch.bfloat16), (3, torch.float32), (5, torch.float16), (8, torch.float32), (8, torch.bfloat16), (4, torch.float64))] + [
    (K, dtype, form) for form in (1, 3) for K, dtype in ((9, torch.bfloat16), (16, torch.bfloat16), (14, torch.float16), (12, torch.float32))]


@pytest.mark.parametrize("K,dtype,form", CASES)
def test_result_and_statistics(K, dtype, form):
    s = Shape(K, dtype, form)
    w = workload(s.sizes, K, dtype, 20 + K)
    stats = [torch.full((w.n_layers, 2), -1.0, dtype=torch.float64, device=DEV) for _ in range(3)]
    outs = []
    for st, wait in zip(stats, (10_000, -1, 1)):
        outs.append(B.adasum_reduce(w.grads, s.offs, layer_stats=st, workspace=s.workspace, resident_wait_us=wait))
        if wait == -1:
            assert s.redone() == s.waiting
    torch.cuda.synchronize()
    for o, st in zip(outs[1:], stats[1:]):
        assert torch.equal(outs[0], o) and torch.equal(stats[0], st)
    out = torch.empty_like(outs[0])
    B.adasum_reduce(w.grads, s.offs, out, noalloc=True, resident_wait_us=-1)
    assert torch.equal(outs[0], out)


@pytest.mark.parametrize("K,dtype,form", [(8, torch.bfloat16, 1), (8, torch.bfloat16, 2), (8, torch.bfloat16, 3), (3, torch.float32, 2)])
def test_after_optimizer_form_in_place(K, dtype, form):
    """A unit that gave up reads `start` again, which other units have written over: each only its own elements."""
    s = Shape(K, dtype, form, delta=True)
    w = W.after_local_step(s.sizes, K, dtype=dtype, device=DEV, seed=12, step=0.25)
    want = B.adasum_reduce(w.grads, s.offs, delta_start=w.meta["start"])
    for wait in (-1, 1):
        got = w.meta["start"].clone()
        B.adasum_reduce(w.grads, s.offs, got, delta_start=got, workspace=s.workspace, resident_wait_us=wait)
        if wait == -1:
            assert s.redone() == s.waiting
        assert torch.equal(want, got)


@pytest.mark.parametrize("K,dtype", [(8, torch.float32), (16, torch.bfloat16)])
def test_left_to_right_order(K, dtype):
    s = Shape(K, dtype, 3)
    w = workload(s.sizes, K, dtype, 30)
    want = B.adasum_reduce(w.grads, s.offs, order=B.ORDER_LINEAR)
    got = B.adasum_reduce(w.grads, s.offs, order=B.ORDER_LINEAR, workspace=s.workspace, resident_wait_us=-1)
    assert s.redone() == s.waiting and torch.equal(want, got)


@pytest.mark.parametrize("layers", [2_000, 20_000])
def test_many_units(layers):
    """More units than 2048 workgroups of the second launch look at four each, and fewer; every tenth layer has two."""
    sizes = [1500 if l % 10 else 2100 for l in range(layers)]
    w = workload(sizes, 3, torch.bfloat16, 4)
    steps, units = steps_and_layers(3, w.layer_offsets, B.BF16)
    assert steps == 1 and units.sum() > layers
    base = B.adasum_workspace_bytes(3, w.layer_offsets, B.BF16, separate_passes=True)
    ws = torch.empty(B.adasum_workspace_bytes(3, w.layer_offsets, B.BF16), dtype=torch.uint8, device=DEV)
    want = B.adasum_reduce(w.grads, w.layer_offsets)
    got = B.adasum_reduce(w.grads, w.layer_offsets, workspace=ws, resident_wait_us=-1)
    assert torch.equal(want, got)
    flags = ws[base:][: 4 * (1 + int(units.sum()))].view(torch.int32)[1:]
    assert int((flags == 2).sum()) == int(units[units > 1].sum())


def test_held_plan_captured_and_replayed():
    """The second launch moves the tag on for the next call whatever it had to do."""
    K, sizes = 4, [3000, 17, 900000, 1]
    w = workload(sizes, K, torch.float32, 5)
    patient, none = (B.Plan(K, w.layer_offsets, torch.float32, resident_wait_us=u) for u in (10_000, -1))
    want, out = torch.empty(w.N, device=DEV), torch.empty(w.N, device=DEV)
    none.execute(w.grads, out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        none.execute(w.grads, out)
    for rep in range(4):
        for i, t in enumerate(w.grads):
            t.mul_(1.0 + 0.5 * ((i + rep) % 3)).add_(0.01 * rep)
        out.fill_(float("nan"))
        g.replay()
        patient.execute(w.grads, want)
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep
        none.execute(w.grads, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep


def test_limits_of_the_option():
    w = workload([5000], 2, torch.float32, 1)
    for bad in (-2, 10_001):
        with pytest.raises(B.AdasumError) as e:
            B.adasum_reduce(w.grads, w.layer_offsets, resident_wait_us=bad)
        assert e.value.code == B.ERR_INVALID_ARG
