"""Translation renders of many workgroups, whose waves take four or eight rows of rays each,
against the same views rendered one at a time, which are few enough for the kernel of single
rows: the same expressions per ray, so the pixels are equal bit for bit. The loss is held to the renders' bound, 1e-5 relative (its FP32 partial sums
take some ten additions each, the rest is FP64).
"""

import pytest
import torch

from paper_2307_03017_amd import hsgd
from tests._problems import rig

pytestmark = pytest.mark.gpu

# (W, H, N): four rows from 192 workgroups of 63 x 16 rays on, eight from 1536 of 63 x 32
SIZES = [(64, 17, 48), (130, 47, 22), (190, 15, 48), (64, 400, 60), (127, 415, 40)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("D", [1, 2, 5, 64])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_many_views_equal_single_ones(size, D, dtype):
    W, H, N = size
    rg = rig(D, N, D, W, H, 0.8 * W, 0.4)       # shifts up to a third of the frame
    gen = torch.Generator(device="cuda").manual_seed(D)
    m = torch.rand((D, H, W, 4), generator=gen, device="cuda").to(dtype)
    images = torch.rand((N, H, W, 3), generator=gen, device="cuda")

    def table(views):
        return hsgd.level_warps(rg["K_ref"], rg["K"][views], rg["R"][views], rg["t"][views], rg["depths"], W, H, W, H)

    every = table(slice(0, N))
    assert every.shift_only
    got, loss = hsgd.hsgd_render(m, every, N, images=images, want_loss=True)
    for i in range(N):
        one, _ = hsgd.hsgd_render(m, table(slice(i, i + 1)), 1)
        assert torch.equal(got[i], one[0]), i
    want = ((got.double() - images.double()) ** 2).sum().item() / (2 * N)
    assert abs(loss.item() - want) <= 1e-5 * want
