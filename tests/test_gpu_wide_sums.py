"""The sums of a wide first pass (radix 32 and 64, the default of 16-bit gradients of more than 16 workers): at most 64
products of whole granules in fp32, everything else in fp64."""
import numpy as np
import pytest
import torch

from paper_2006_02924_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("R", [32, 64])
def test_constant_layers(R, dtype):
    """Equal addends round the same way throughout a binade, so the error of a long fp32 sum grows with its length: a
    wave's share of the long layer's spans has 65536 products.  64 additions in fp32 err by at most 63 * 2^-24."""
    print(f"constant layers R={R} {dtype}", flush=True)
    offs = [0, 1 << 27, (1 << 27) + 4099]
    values = [1 + k / 128 for k in (53, 89, 101)]
    bufs = [torch.full((offs[-1],), v, dtype=dtype, device=DEV) for v in values]
    gram = B.adasum_group_gram([bufs[r % 3] for r in range(R)], offs).cpu().numpy()
    v = np.array([values[r % 3] for r in range(R)])
    for l in range(2):
        want = np.outer(v, v) * (offs[l + 1] - offs[l])
        assert np.max(np.abs(gram[l] - want) / want) <= 63 * 2.0 ** -24


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("R", [32, 64])
def test_ragged_elements_are_summed_in_64_bits(R, dtype):
    """Layers that are all head and tail (no eight elements on the granule grid)."""
    print(f"ragged layers R={R} {dtype}", flush=True)
    offs = [0, 1, 15, 16, 29, 32, 32, 46, 8192 * 3 - 7, 8192 * 3 + 7]
    gen = torch.Generator(device=DEV).manual_seed(3)
    x = torch.randn(R, offs[-1], device=DEV, generator=gen) * 10.0 ** (torch.rand(1, offs[-1], device=DEV, generator=gen) * 3 - 1.5)
    x = x.to(dtype)
    gram = B.adasum_group_gram([row.clone() for row in x], offs).cpu().numpy()
    rows = x.double().cpu().numpy()
    for l, (lo, hi) in enumerate(zip(offs, offs[1:])):
        part = rows[:, lo:hi]
        bound = np.abs(part) @ np.abs(part).T
        whole = max(0, hi // 8 * 8 - (lo + 7) // 8 * 8)
        eps = 2.0 ** -48 if whole == 0 else 63 * 2.0 ** -24
        assert np.all(np.abs(gram[l] - part @ part.T) <= eps * bound), l


@pytest.mark.parametrize("R", [32, 64])
def test_layers_of_many_spans(R):
    """Around the number of spans (of 2048 elements here) from which a layer's are folded in runs of 16 first."""
    print(f"many spans R={R}", flush=True)
    offs = np.cumsum([0, 5, 32 * 2048 - 5, 33 * 2048, 48 * 2048 + 9, 2048 * 3 - 9, 65 * 2048, 17 * 2048]).tolist()
    gen = torch.Generator(device=DEV).manual_seed(5)
    x = (torch.randn(R, offs[-1], device=DEV, generator=gen) + 0.25).to(torch.bfloat16)
    gram = B.adasum_group_gram([row.clone() for row in x], offs)
    for l, (lo, hi) in enumerate(zip(offs, offs[1:])):
        part = x[:, lo:hi].double()
        assert torch.all((gram[l] - part @ part.T).abs() <= 63 * 2.0 ** -24 * (part.abs() @ part.abs().T)), l
