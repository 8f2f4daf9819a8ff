"""What a plan's resident pass looks like from outside: its units, from the bytes its section adds to the workspace."""
import numpy as np

from paper_2006_02924_amd import binding as B

LANES = 256                                   # granules of a step
SLOTS = {1: 768, 2: 768, 3: 512}              # workgroups on the chip (form 1 of more than 8 16-bit operands: 512)


def up(n, a):
    return (n + a - 1) // a * a


def operands(K):
    return K if K <= 8 else (K + 1) // 2 * 2


def unit_count(K, offs, code, **kw):
    """Units of the resident pass, 0 where the other passes are taken (a reduction of a single pass)."""
    need, base = (B.adasum_workspace_bytes(K, offs, code, separate_passes=s, **kw) for s in (False, True))
    if need == base:
        return 0
    words = operands(K) * (operands(K) + 1)       # two per entry of the Gram matrix
    size = lambda n: up(4 * (1 + n), 256) + up((n + len(offs) - 1) * words * 8, 256)
    n = max(1, (need - base - 1024) // (words * 8 + 4) - (len(offs) - 1))
    while size(n) < need - base:
        n += 1
    found = [m for m in range(max(1, n - 40), n + 40) if size(m) == need - base]
    assert found, (need, base)
    return found


def steps_and_layers(K, offs, code, **kw):
    """Steps of a unit and the units of every layer."""
    vec = {B.F32: 4, B.BF16: 8, B.F16: 8, B.F64: 2}[code]
    found = unit_count(K, offs, code, **kw)
    assert found, "not taken as a resident pass"
    for n in range(1, 33):
        layers = B.plan_tiles(offs, LANES * vec * n)["layer"]
        if len(layers) in found:
            return n, np.bincount(layers, minlength=len(offs) - 1)
    raise AssertionError(found)
