"""Which reductions are taken as a resident pass, as far as the host decides it (no GPU needed)."""
import ctypes as C

import pytest

from paper_2006_02924_amd import binding as B
from paper_2006_02924_amd import workloads as W
from tests.resident_util import steps_and_layers, unit_count


def noalloc(lib, K, offs, dtype):
    """adasum_reduce_noalloc with addresses that are never used: what the host makes of the sizes."""
    o = B.Options()
    o.struct_bytes = C.sizeof(B.Options)
    o.out_dtype = -1
    grads = (C.c_void_p * K)(*[C.c_void_p((k + 1) << 40) for k in range(K)])
    table = (C.c_int64 * len(offs))(*offs)
    return lib.adasum_reduce_noalloc(grads, K, table, len(offs) - 1, dtype, C.c_void_p((K + 1) << 40), C.byref(o), None)


@pytest.mark.parametrize("K,dtype,sizes,resident", [
    (16, B.BF16, [3_000] * 8_000, False), (16, B.BF16, [2_360_000] * 100, False), (16, B.F32, [1_400_000] * 80, False),
    (16, B.BF16, [3_000] * 4_000, True), (8, B.F32, [1_000_000] * 25, True)])
def test_the_resident_pass_is_taken_by_every_entry_point_or_none(K, dtype, sizes, resident):
    """Where the other passes fit the scratch of the entry point without allocation and the resident pass does not, the
    plans and the workspace of the other entry points are without it too: all of them give the same bits."""
    offs = W.offsets_from_sizes(sizes)
    need, without = (B.adasum_workspace_bytes(K, offs, dtype, separate_passes=s) for s in (False, True))
    assert (need > without) == resident
    assert need < B.NOALLOC_SCRATCH_BYTES


@pytest.mark.parametrize("K,dtype,sizes", [(2, B.F32, [3_000_000] * 1_500), (2, B.F64, [3_000_000] * 900)])
def test_what_fits_without_allocation_does_not_depend_on_the_route(lib, K, dtype, sizes):
    """The tables of a resident pass are the smaller ones here and would fit; those of the other passes do not."""
    assert noalloc(lib, K, W.offsets_from_sizes(sizes), dtype) == B.ERR_TOO_LARGE


def steps(K, sizes, dtype, **kw):
    return steps_and_layers(K, W.offsets_from_sizes(sizes), dtype, **kw)


def test_units_are_as_small_as_the_chip_holds_at_once():
    # (one granule a lane: at most half of 768 for one layer)
    n, units = steps(2, [384 * 2048], B.BF16)
    assert (n, units.max()) == (1, 384)
    n, units = steps(2, [900_000], B.BF16)
    assert n == 2 and units.max() == 220
    n, units = steps(2, [10_000_000], B.BF16)
    assert units.max() <= 384 and 1 < n < 18
    n, units = steps(2, [10_000_000] * 5, B.BF16)
    assert n == 18 and units.sum() > 768
    # more than 8 operands of a 16-bit type: 512 workgroups, 256 for one layer
    n, units = steps(12, [250_000, 250_000, 500_000], B.BF16)
    assert (n, units.sum()) == (1, 491)
    n, units = steps(12, [250_000, 250_000, 600_000], B.BF16)
    assert n == 2
    n, units = steps(12, [250_000] * 7, B.F32)
    assert n == 3 and units.sum() > 512


def test_tables_of_tiny_layers_take_the_smallest_units():
    assert steps(2, [200] * 20_000, B.BF16)[0] == 1
    assert steps(8, [700] * 4_000, B.F64)[0] == 1
    assert unit_count(16, W.offsets_from_sizes([6145] * 700), B.BF16)[0] > 2 * 700      # (three or four units of one step each)
    crossing = [2048 * 2 - 8] * 600                                                    # 2 .. 3 units of one step, 1 .. 2 of four
    assert len(B.plan_tiles(W.offsets_from_sizes(crossing), 4 * 2048)) in unit_count(9, W.offsets_from_sizes(crossing), B.BF16)
    assert len(B.plan_tiles(W.offsets_from_sizes(crossing), 2048)) in unit_count(12, W.offsets_from_sizes(crossing), B.BF16)
    assert steps(2, [200] * 2_000 + [3_000_000], B.BF16)[0] > 1        # (a layer that would have 1465 of them)


@pytest.mark.parametrize("K,dtype,unit", [(16, B.F32, 3072), (16, B.BF16, 6144), (2, B.BF16, 24 * 2048)])
def test_many_layers_that_each_leave_the_chip_half_idle_take_the_other_passes(K, dtype, unit):
    assert unit_count(K, W.offsets_from_sizes([300 * unit] * 5), dtype) == 0
    assert unit_count(K, W.offsets_from_sizes([300 * unit] * 4), dtype)
    assert unit_count(K, W.offsets_from_sizes([200 * unit] * 5), dtype)
    assert unit_count(K, W.offsets_from_sizes([(470 if dtype == B.F32 else 400) * unit] * 5), dtype)
    assert bool(unit_count(K, W.offsets_from_sizes([400 * unit] * 5), dtype)) == (dtype != B.F32)
    assert unit_count(K, W.offsets_from_sizes([300 * unit] * 5 + [200 * unit] * 9), dtype)


def test_fp32_of_few_rows_stays():
    assert unit_count(8, W.offsets_from_sizes([300 * 7168] * 20), B.F32)


def test_the_wait_option(lib):
    """Values out of range and the reserved word are refused; a struct that ends before them reads as 0."""
    def call(**fields):
        o = B.Options()
        o.struct_bytes = C.sizeof(B.Options)
        o.out_dtype = -1
        for k, v in fields.items():
            setattr(o, k, v)
        grads = (C.c_void_p * 2)(C.c_void_p(1 << 40), C.c_void_p(2 << 40))
        return lib.adasum_reduce_ex(grads, 2, (C.c_int64 * 1)(0), 0, B.F32, C.c_void_p(3 << 40), C.byref(o), None)

    for us in (0, 1, 10_000, -1):
        assert call(resident_wait_us=us) == B.OK
    for bad in ({"resident_wait_us": -2}, {"resident_wait_us": 10_001}, {"reserved2": 1}):
        assert call(**bad) == B.ERR_INVALID_ARG
        assert call(struct_bytes=B.Options.resident_wait_us.offset, **bad) == B.OK
    assert call(struct_bytes=B.Options.resident_wait_us.offset, reserved1=1) == B.ERR_INVALID_ARG
