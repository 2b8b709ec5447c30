"""General homographies with more planes than 32: masks and ranks in both halves of a mask word,
the last plane of 64, dense gradients of the kernel's larger form, odd plane counts at its end.
Bounds as for fewer planes: a composite of D planes 10 (D + 2) 2^-24; a gradient entry 4 times
that and 2^-24 per view and tap summed, relative to the largest entry and to the whole.
"""

import numpy as np
import pytest
import torch

from oracle import hsgd_oracle as O
from paper_2307_03017_amd import hsgd
from tests._problems import device_warps, f32, mask_bits, oracle_maps, rel_err, rig

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("size", [(65, 5), (131, 37)], ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("D,k", [(34, 33), (63, 5), (63, None), (64, 1), (64, 40), (64, 63), (64, None)])
def test_render_and_gradient(D, k, size, dtype):
    W, H = size
    rg = rig(D, 2, D, W, H, 0.8 * W, 0.1, general=True)
    rng = np.random.default_rng(D * 1000 + W)
    M, I = f32(rng.uniform(size=(D, H, W, 4))), f32(rng.uniform(size=(2, H, W, 3)))
    M[..., 3] **= 6                            # light reaches the far planes
    M = O.bf16_round(M) if dtype == torch.bfloat16 else f32(M)
    G = oracle_maps(O, rg)
    table, Md = device_warps(hsgd, rg), torch.from_numpy(M.astype(np.float32)).cuda().to(dtype)
    images = torch.from_numpy(I.astype(np.float32)).cuda()
    out, _ = hsgd.hsgd_render(Md, table, 2)
    assert np.abs(out.cpu().numpy() - O.render(M, G)).max() <= 10 * (D + 2) * EPS
    want_loss, ref = O.loss_and_grad(M, G, I)
    mask = hsgd.hsgd_select_active(Md, k, with_ids=False) if k else None
    if k:
        ref = np.where(mask_bits(mask.cpu().numpy(), D)[..., None], ref, 0.0)
    assert ref[-1].any() or (k and k < 33)     # the last plane takes part where many are kept
    g, loss = hsgd.hsgd_grad_step(Md, table, 2, images=images, mask=mask, kcap=k, want_grad=True, want_loss=True)
    g = g.cpu().numpy()
    bound = (40 * (D + 2) + 8) * EPS
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    assert rel_err(g, ref) <= bound and np.abs(g - ref).max() <= bound * np.abs(ref).max()
