"""A large tilted FP32 plane sweep whose second level goes through the caches (64 MiB at the first,
rows that end inside a write request), bit for bit against its views one at a time, whose volumes
are small enough to stream.
"""

import pytest
import torch

from paper_2307_03017_amd import hsgd
from tests._problems import rig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,L", [(366, 250, 2), (388, 236, 3), (390, 234, 2)])
def test_equal_to_single_views(W, H, L):
    N, D = 2, 32
    assert N * D * W * H * 12 >= 64 << 20 > D * W * H * 12 and W // 2 * 12 % 64
    rg = rig(W, N, D, W, H, 0.8 * W, 0.1, general=True)
    images = torch.rand((N, H, W, 3), generator=torch.Generator(device="cuda").manual_seed(W), device="cuda")

    def sweep(views):
        table = hsgd.psv_warps(rg["K_ref"], rg["K"][views], rg["R"][views], rg["t"][views], rg["depths"])
        assert not table.shift_only
        return hsgd.hsgd_plane_sweep(images[views], table, D, L)

    every = sweep(slice(0, N))
    for i in range(N):
        for got, want in zip(every, sweep(slice(i, i + 1))):
            assert torch.equal(got[i], want[0])
