"""Translation renders of several rows of rays per wave at the sizes where that begins: the same
pixels, bit for bit, as one view at a time by the kernel of single rows; one view alone, which has
no such call beside it, against the oracle (a sample is off by ~10 roundings of numbers up to 1, a
composite by those of its D planes: 10 (D + 2) 2^-24).
"""

import numpy as np
import pytest
import torch

from oracle import hsgd_oracle as O
from paper_2307_03017_amd import hsgd
from tests._problems import oracle_maps, rig

pytestmark = pytest.mark.gpu


def rows_of(D, H, W, N):
    return hsgd.lib()["_ZN4hsgd11render_rowsEiiii"](D, H, W, N)


def problem(W, H, D, N, dtype):
    rg = rig(D, N, D, W, H, 0.8 * W, 0.4)
    gen = torch.Generator(device="cuda").manual_seed(D)
    return rg, torch.rand((D, H, W, 4), generator=gen, device="cuda").to(dtype), torch.rand((N, H, W, 3), generator=gen, device="cuda")


def table(rg, views):
    return hsgd.level_warps(rg["K_ref"], rg["K"][views], rg["R"][views], rg["t"][views], rg["depths"], rg["W"], rg["H"],
                            rg["W"], rg["H"])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("rows,size", [(4, (190, 47, 1, 64)), (4, (190, 47, 5, 64)), (4, (64, 63, 16, 64)), (4, (130, 47, 64, 64)),
                                       (4, (700, 130, 17, 4)), (8, (127, 415, 2, 40))], ids=str)
def test_equal_to_single_rows(rows, size, dtype):
    W, H, D, N = size
    assert rows_of(D, H, W, N) == rows and rows_of(D, H, W, 1) == 1
    rg, m, images = problem(W, H, D, N, dtype)
    got, loss = hsgd.hsgd_render(m, table(rg, slice(0, N)), N, images=images, want_loss=True)
    for i in range(N):
        assert torch.equal(got[i], hsgd.hsgd_render(m, table(rg, slice(i, i + 1)), 1)[0][0]), i
    want = ((got.double() - images.double()) ** 2).sum().item() / (2 * N)
    assert abs(loss.item() - want) <= 1e-5 * want


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
def test_one_view(dtype):
    W, H, D = 640, 250, 24
    assert rows_of(D, H, W, 1) == 4
    rg, m, _ = problem(W, H, D, 1, dtype)
    got, _ = hsgd.hsgd_render(m, table(rg, slice(0, 1)), 1)
    want = O.render(m.float().cpu().numpy().astype(np.float64), oracle_maps(O, rg))
    assert np.abs(got.cpu().numpy() - want).max() <= 10 * (D + 2) * 2.0 ** -24
