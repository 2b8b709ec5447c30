"""General homographies at the sizes and rigs where their kernels branch: frames smaller than,
equal to and just over a wave's row and a workgroup's tile, plane counts around the blocks the
kernels step in, and rigs whose samples leave the plane, rotate across it, zoom or pass behind
the camera.

Bounds. Positions are FP64 and only the fractions are rounded, so a sample is off by a few
roundings of numbers up to 1 (fractions, weights, four FMAs: ~10) and a composite by those of
its D planes: 10 (D + 2) 2^-24. A gradient entry is a sum of such products: relative to the
whole gradient the same bound, with a factor 4 for the differences of colours in its alpha
channel and 2^-24 per view and tap summed.
"""

import numpy as np
import pytest
import torch

from oracle import hsgd_oracle as O
from paper_2307_03017_amd import hsgd, scenes
from tests._problems import device_warps, f32, mask_bits, oracle_maps, rel_err, rot

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
SIZES = [(2, 2), (5, 65), (65, 5), (64, 16), (131, 37)]
RIGS = ["tilt", "roll", "zoom", "behind", "mixed"]


def make_rig(kind, N, D, W, H):
    rng = np.random.default_rng(sum(map(ord, kind)) + W)
    f = 0.8 * W
    K = np.array([[f, 0.0, (W - 1) / 2.0], [0.0, f, (H - 1) / 2.0], [0.0, 0.0, 1.0]])
    Ks = np.repeat(K[None], N, axis=0)
    t = np.concatenate([rng.uniform(-0.1, 0.1, (N, 2)), rng.uniform(-0.03, 0.03, (N, 1))], axis=1)
    R = np.stack([rot(*(rng.normal(size=3) * 0.02)) for _ in range(N)])
    if kind == "roll":
        R = np.stack([rot(0.01, 0.02, 0.7 + 0.9 * i) for i in range(N)])
    elif kind == "zoom":
        Ks = np.stack([np.diag([s, s, 1.0]) @ K for s in (0.45, 2.2)[:N]])
    elif kind == "behind":
        R = np.stack([rot(0.1, 1.25 * (-1) ** i, 0.05) for i in range(N)])
    elif kind == "mixed":                       # one translating view among rotating ones
        R[0] = np.eye(3)
        t[0, 2] = 0.0
    return dict(K_ref=K, K=Ks, R=R, t=t, depths=scenes.plane_depths(D), W=W, H=H)


def problem(kind, N, D, W, H):
    rng = np.random.default_rng(D * 1000 + W)
    return make_rig(kind, N, D, W, H), f32(rng.uniform(0.05, 0.95, size=(D, H, W, 4))), f32(rng.uniform(size=(N, H, W, 3)))


def dev(x, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda().to(dtype)


@pytest.mark.parametrize("kind", RIGS)
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("D", [1, 4, 33])
def test_render_matches_oracle(kind, size, D):
    W, H = size
    rg, M, I = problem(kind, 2, D, W, H)
    G = oracle_maps(O, rg)
    for dtype in (torch.float32, torch.bfloat16):
        Ms = O.bf16_round(M) if dtype == torch.bfloat16 else M
        ref = O.render(Ms, G)
        out, loss = hsgd.hsgd_render(dev(M, dtype), device_warps(hsgd, rg), 2, images=dev(I), want_loss=True)
        assert np.abs(out.cpu().numpy() - ref).max() <= 10 * (D + 2) * EPS
        want = O.photometric_loss(ref, I)
        assert abs(loss.item() - want) <= 1e-5 * want


@pytest.mark.parametrize("kind", RIGS)
@pytest.mark.parametrize("size,L", [((2, 2), 1), ((66, 6), 2), ((64, 16), 5), ((132, 36), 3)],
                         ids=lambda s: f"{s[0]}x{s[1]}" if isinstance(s, tuple) else f"L{s}")
def test_plane_sweep_matches_oracle(kind, size, L):
    W, H = size
    rg, _, I = problem(kind, 2, 5, W, H)
    ref = O.psv_pyramid(O.plane_sweep(I, rg["K_ref"], rg["K"], rg["R"], rg["t"], rg["depths"]), L)
    table = hsgd.psv_warps(rg["K_ref"], rg["K"], rg["R"], rg["t"], rg["depths"])
    out = hsgd.hsgd_plane_sweep(dev(I), table, 5, L)
    half = hsgd.hsgd_plane_sweep(dev(I), table, 5, L, dtype=torch.bfloat16)
    for want, got, b in zip(ref, out, half):
        assert np.abs(got.cpu().numpy() - want).max() <= 20 * EPS
        assert torch.equal(b, got.to(torch.bfloat16))


@pytest.mark.parametrize("kind", RIGS)
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("D,k", [(1, 1), (4, 2), (5, None), (33, 4)])
def test_gradient_matches_oracle(kind, size, D, k):
    """k planes of each pixel selected, or every voxel (None), in both storages."""
    W, H = size
    rg, M, I = problem(kind, 2, D, W, H)
    G = oracle_maps(O, rg)
    for dtype in (torch.float32, torch.bfloat16):
        Ms = O.bf16_round(M) if dtype == torch.bfloat16 else M
        want_loss, ref = O.loss_and_grad(Ms, G, I)
        Md = dev(M, dtype)
        mask = None
        if k:
            mask = hsgd.hsgd_select_active(Md, k, with_ids=False)
            ref = np.where(mask_bits(mask.cpu().numpy(), D)[..., None], ref, 0.0)
        g, loss = hsgd.hsgd_grad_step(Md, device_warps(hsgd, rg), 2, images=dev(I), mask=mask, kcap=k,
                                      want_grad=True, want_loss=True)
        assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
        bound = (40 * (D + 2) + 8) * EPS
        got = g.cpu().numpy()
        assert rel_err(got, ref) <= bound
        assert np.abs(got - ref).max() <= bound * max(np.abs(ref).max(), 1e-30)
