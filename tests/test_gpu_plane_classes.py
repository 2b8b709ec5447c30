"""Plane counts at the edges of the classes that the translation-path kernels are compiled
for (8, 16, 24, 32, 40, 48, 64), where the last class's planes end or a new class begins.

The gradient and the render are held to the FP64 oracle at the parity bounds (1e-4 relative,
1e-5 absolute), the selection is exact, and a refinement (fused upsampling and selection, by
pixel on small levels and by 2 x 2 blocks on large ones) equals the same steps taken one
call at a time bit for bit: every voxel goes through the same expressions.
"""

import numpy as np
import pytest
import torch

from oracle import hsgd_oracle as O
from paper_2307_03017_amd import hsgd
from tests._problems import device_warps, f32, grad_close, mask_bits, oracle_maps, rig

pytestmark = pytest.mark.gpu

PLANES = [17, 24, 25, 33, 40, 41, 48, 49]
DTYPES = [torch.float32, torch.bfloat16]


def dev(x, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda().to(dtype)


@pytest.mark.parametrize("dtype", DTYPES, ids=["fp32", "bf16"])
@pytest.mark.parametrize("D", PLANES)
def test_gradient_render_and_selection_match_oracle(D, dtype):
    W, H, N, k = 75, 23, 2, 3
    rng = np.random.default_rng(D)
    rg = rig(D, N, D, W, H, 50.0, 0.1)
    M = f32(rng.uniform(0.05, 0.95, size=(D, H, W, 4)))
    I = f32(rng.uniform(size=(N, H, W, 3)))
    Ms = O.bf16_round(M) if dtype == torch.bfloat16 else M
    G = oracle_maps(O, rg)
    Md, table = dev(M, dtype), device_warps(hsgd, rg)
    out, _ = hsgd.hsgd_render(Md, table, N)
    assert np.abs(out.cpu().numpy() - O.render(Ms, G)).max() <= 1e-5
    _, want = O.loss_and_grad(Ms, G, I)
    g, _ = hsgd.hsgd_grad_step(Md, table, N, images=dev(I), want_grad=True)
    grad_close(g.cpu().numpy(), want, 1e-4, "dense")
    mask = hsgd.hsgd_select_active(Md, k, with_ids=False)
    S = mask_bits(mask.cpu().numpy(), D)
    assert np.array_equal(S, O.select_active(Ms[..., 3], k))
    g, _ = hsgd.hsgd_grad_step(Md, table, N, images=dev(I), mask=mask, kcap=k, want_grad=True)
    g = g.cpu().numpy()
    assert np.all(g[~S] == 0.0)
    grad_close(g[S], want[S], 1e-4, "restricted")


@pytest.mark.parametrize("dtype", DTYPES, ids=["fp32", "bf16"])
@pytest.mark.parametrize("size", [(66, 36), (248, 2048)], ids=["by pixel", "by block"])
@pytest.mark.parametrize("D", [7, 16, 24, 40, 41, 48])
def test_refinement_equals_its_steps(D, size, dtype):
    W, H = size
    N, k, lr = 2, 3, 0.5
    rg = rig(D, N, D, W, H, 0.8 * W, 0.1)
    gen = torch.Generator(device="cuda").manual_seed(D)
    images = torch.rand((N, H, W, 3), generator=gen, device="cuda")
    m = torch.rand((D, H // 2, W // 2, 4), generator=gen, device="cuda").to(dtype)
    got, _ = hsgd.hsgd_refine(m, images, rg["K_ref"], rg["K"], rg["R"], rg["t"], rg["depths"], [1, 1], k,
                              lr_rgb=lr, lr_alpha=lr)
    small = hsgd.hsgd_downsample2x(images)
    for level, target in enumerate([small, images]):
        if level:
            m = hsgd.hsgd_upsample2x(m)
        mask = hsgd.hsgd_select_active(m, k, with_ids=False)
        table = device_warps(hsgd, rg, m.shape[2], m.shape[1])
        hsgd.hsgd_grad_step(m, table, N, images=target, mask=mask, kcap=k, lr_rgb=lr, lr_alpha=lr)
    assert torch.equal(got, m)
