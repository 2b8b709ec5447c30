"""General homographies with few planes: the renderer's form for one and two, and every remainder
of the groups in which planes are fetched ahead, in the renderer and the gradient. Bounds as for
other plane counts: a composite of D planes 10 (D + 2) 2^-24; a gradient entry 4 times that and
2^-24 per view and tap summed, relative to the largest entry.
"""

import numpy as np
import pytest
import torch

from oracle import hsgd_oracle as O
from paper_2307_03017_amd import hsgd
from tests._problems import device_warps, f32, oracle_maps, rig

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
W, H, N = 67, 11, 2


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("kind", ["tilted", "mixed"])
@pytest.mark.parametrize("D", [1, 2, 3, 5, 6, 7, 8, 9])
def test_render_and_gradient(D, kind, dtype):
    rg = rig(D, N, D, W, H, 0.8 * W, 0.1, general=True)
    if kind == "mixed":                        # one translating view beside a tilted one
        rg["R"][0], rg["t"][0, 2] = np.eye(3), 0.0
    rng = np.random.default_rng(D)
    M, I = f32(rng.uniform(0.05, 0.95, size=(D, H, W, 4))), f32(rng.uniform(size=(N, H, W, 3)))
    M = O.bf16_round(M) if dtype == torch.bfloat16 else M
    G, table = oracle_maps(O, rg), device_warps(hsgd, rg)
    assert not table.shift_only
    Md = torch.from_numpy(M.astype(np.float32)).cuda().to(dtype)
    images = torch.from_numpy(I.astype(np.float32)).cuda()
    out, loss = hsgd.hsgd_render(Md, table, N, images=images, want_loss=True)
    want_loss, ref = O.loss_and_grad(M, G, I)
    assert np.abs(out.cpu().numpy() - O.render(M, G)).max() <= 10 * (D + 2) * EPS
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    g, loss = hsgd.hsgd_grad_step(Md, table, N, images=images, want_grad=True, want_loss=True)
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    assert np.abs(g.cpu().numpy() - ref).max() <= (40 * (D + 2) + 8) * EPS * np.abs(ref).max()
