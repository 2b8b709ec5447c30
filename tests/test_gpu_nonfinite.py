"""Values that are no numbers, in maps and planes of the general kernels: what the zero padding
and the ray's frame exclude stays excluded, whatever the excluded numbers are.

Bounds as for finite maps: a composite of D planes 10 (D + 2) 2^-24, a gradient entry 4 times
that and 2^-24 per view and tap summed, relative to the largest entry.
"""

import numpy as np
import pytest
import torch

from oracle import hsgd_oracle as O
from paper_2307_03017_amd import hsgd
from tests._problems import f32, mask_bits, rig

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
N, D, W, H = 2, 3, 70, 20


def dev(x, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda().to(dtype)


def records():
    """A tilted rig's map records as writable bytes and their G as [N][D][3][3]."""
    rg = rig(3, N, D, W, H, 0.8 * W, 0.05, general=True)
    raw = hsgd.hsgd_build_warps(rg["K_ref"], rg["K"], rg["R"], rg["t"], rg["depths"])
    assert not any(r.is_shift for r in hsgd.warp_records(raw))
    return raw, raw.view(np.float64)[:, :, :9].reshape(N, D, 3, 3)


INF, NAN = np.inf, np.nan
# entries of one plane's map: a position that is no number lies outside the plane, one at a
# finite point over an infinite depth at the corner
MAPS = {
    "nan_scale": {(0, 0): NAN}, "nan_offset": {(1, 2): NAN}, "nan_depth": {(2, 2): NAN},
    "inf_scale": {(0, 0): INF}, "minus_inf_offset": {(1, 2): -INF}, "inf_skew": {(0, 1): -INF},
    "inf_depth": {(2, 2): INF}, "inf_over_inf": {(0, 2): INF, (2, 2): INF}, "nan_row": {(0, 0): NAN, (1, 1): NAN},
    "tiny_depth": {(0, 2): 1.0, (1, 2): 1.0, (2, 0): 0.0, (2, 1): 0.0, (2, 2): 1e-310},
}


def broken(name):
    raw, G = records()
    for view, plane in ((0, 1), (1, 2)):
        for (r, c), v in MAPS[name].items():
            raw[view, plane, (3 * r + c) * 8:(3 * r + c + 1) * 8] = np.frombuffer(np.float64(v).tobytes(), np.uint8)
    return hsgd.WarpTable(raw), raw.view(np.float64)[:, :, :9].reshape(N, D, 3, 3)


@pytest.mark.parametrize("name", MAPS)
def test_render_and_gradient_under_maps_that_are_no_numbers(name):
    table, G = broken(name)
    assert not table.shift_only
    rng = np.random.default_rng(5)
    M, I = f32(rng.uniform(0.05, 0.95, size=(D, H, W, 4))), f32(rng.uniform(size=(N, H, W, 3)))
    with np.errstate(all="ignore"):
        image = O.render(M, G)
        want_loss, ref = O.loss_and_grad(M, G, I)
    out, loss = hsgd.hsgd_render(dev(M), table, N, images=dev(I), want_loss=True)
    assert np.abs(out.cpu().numpy() - image).max() <= 10 * (D + 2) * EPS
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    mask = hsgd.hsgd_select_active(dev(M), 2, with_ids=False)
    for m, k, r in ((None, None, ref), (mask, 2, np.where(mask_bits(mask.cpu().numpy(), D)[..., None], ref, 0.0))):
        g, loss = hsgd.hsgd_grad_step(dev(M), table, N, images=dev(I), mask=m, kcap=k, want_grad=True, want_loss=True)
        assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
        assert np.abs(g.cpu().numpy() - r).max() <= (40 * (D + 2) + 8) * EPS * np.abs(r).max()


@pytest.mark.parametrize("name", MAPS)
def test_plane_sweep_under_maps_that_are_no_numbers(name):
    table, G = broken(name)
    I = f32(np.random.default_rng(6).uniform(size=(N, H, W, 3)))
    with np.errstate(all="ignore"):
        want = np.stack([np.stack([O.sample_bilinear(I[i], G[i, z]) for z in range(D)]) for i in range(N)])
    got, = hsgd.hsgd_plane_sweep(dev(I), table, D, 1)
    assert np.abs(got.cpu().numpy() - want).max() <= 10 * EPS


@pytest.mark.parametrize("bad", [INF, -INF, NAN])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("k", [None, 2])
def test_voxels_that_no_ray_of_the_frame_reads(k, dtype, bad):
    """A shift by (-3.3, -2.4) under the general kernels: only rays past the frame's right and
    lower edge would read the last columns and rows. They have no image, so whatever is stored
    there, the gradient is what it is with ordinary numbers there, and zero in those cells."""
    raw, _ = records()
    G = np.tile(np.eye(3), (N, D, 1, 1))
    G[..., 0, 2], G[..., 1, 2] = -3.3, -2.4
    raw.view(np.float64)[:, :, :9] = G.reshape(N, D, 9)
    table = hsgd.WarpTable(raw)
    assert not table.shift_only
    rng = np.random.default_rng(7)
    M, I = f32(rng.uniform(0.05, 0.95, size=(D, H, W, 4))), f32(rng.uniform(size=(N, H, W, 3)))
    if dtype == torch.bfloat16:
        M = O.bf16_round(M)
    want_loss, ref = O.loss_and_grad(M, G, I)
    mask = hsgd.hsgd_select_active(dev(M, dtype), k, with_ids=False) if k else None
    if k:
        ref = np.where(mask_bits(mask.cpu().numpy(), D)[..., None], ref, 0.0)
    unread = np.zeros((D, H, W), bool)
    unread[:, :, W - 3:] = unread[:, H - 2:] = True
    assert not ref[unread].any()
    Md = dev(np.where(unread[..., None], bad, M), dtype)
    g, loss = hsgd.hsgd_grad_step(Md, table, N, images=dev(I), mask=mask, kcap=k, want_grad=True, want_loss=True)
    g = g.cpu().numpy()
    assert abs(loss.item() - want_loss) <= 1e-5 * want_loss
    assert not g[unread].any()
    assert np.abs(g - ref).max() <= (40 * (D + 2) + 8) * EPS * np.abs(ref).max()


def test_taps_of_no_weight_take_nothing():
    """A position a billionth left of and above a pixel: its fractions round to 1, so the pixel
    itself has all the weight and the three cells beside it none. An infinite upstream value of
    one ray reaches its own cell alone."""
    raw, _ = records()
    G = np.tile(np.eye(3), (N, D, 1, 1))
    G[..., 0, 2] = G[..., 1, 2] = -1e-9
    raw.view(np.float64)[:, :, :9] = G.reshape(N, D, 9)
    table = hsgd.WarpTable(raw)
    rng = np.random.default_rng(8)
    M, up = dev(f32(rng.uniform(0.05, 0.95, size=(D, H, W, 4)))), dev(f32(rng.normal(size=(N, H, W, 3))))
    cells = [(9, 11), (8, 62), (15, 40), (16, 63)]         # inside a tile and at its seams
    for y, x in cells:
        up[0, y, x] = 0.0
    want, _ = hsgd.hsgd_grad_step(M, table, N, dimg=up, want_grad=True)
    for y, x in cells:
        up[0, y, x] = INF
    got, _ = hsgd.hsgd_grad_step(M, table, N, dimg=up, want_grad=True)
    rest = torch.ones((H, W), dtype=torch.bool, device="cuda")
    for y, x in cells:
        rest[y, x] = False
        assert not torch.isfinite(got[:, y, x]).any()
    assert torch.equal(got[:, rest], want[:, rest])
