"""Calls whose workgroups are 2^32 threads or more in all, which is more than one grid dimension
holds (the runtime launches the low 32 bits of the product): long, narrow frames (2 columns in
tiles of 62 to 64), and a conversion of as many values. Identity maps and one plane, so that a
pixel's colour and gradient are its own voxel's: with weight 1 on one tap and 0 on the others
a sample is the voxel exactly, a colour one product; a gradient entry is at most three products
of numbers up to 1 and their sums over two views (8 roundings of values up to 6).
"""

import numpy as np
import pytest
import torch

from paper_2307_03017_amd import hsgd

pytestmark = pytest.mark.gpu

W, H, N = 2, 1 << 25, 2
BOUND = 8 * 6 * 2.0 ** -24


def problem():
    eye = np.eye(3)                           # the reference's own camera, N times
    cameras = eye, np.stack([eye] * N), np.stack([eye] * N), np.zeros((N, 3)), np.ones(1)
    table = hsgd.level_warps(*cameras, W, H, W, H)
    gen = torch.Generator(device="cuda").manual_seed(1)
    m = torch.rand((1, H, W, 4), generator=gen, device="cuda") * 0.5 + 0.25
    images = torch.rand((N, H, W, 3), generator=gen, device="cuda")
    return cameras, table, m, images


def gradient(m, images):
    c, a = m[0, ..., :3], m[0, ..., 3:]
    r = sum(a * c - i for i in images) / N
    return torch.cat([r * a, (r * c).sum(-1, keepdim=True)], dim=-1)[None]


def squares(m, images):
    colour = m[0, ..., 3:] * m[0, ..., :3]
    return sum(((colour - i).double() ** 2).sum().item() for i in images) / (2 * N)


def test_general_render_and_gradient():
    _, table, m, images = problem()
    maps = table.tensor                       # bare records: the general kernels
    out, loss = hsgd.hsgd_render(m, maps, N, images=images, want_loss=True)
    want = m[0, ..., 3:] * m[0, ..., :3]
    assert all(torch.equal(o, want) for o in out)
    total = squares(m, images)
    assert abs(loss.item() - total) <= 1e-5 * total
    del out, want
    g, loss = hsgd.hsgd_grad_step(m, maps, N, images=images, want_grad=True, want_loss=True)
    assert abs(loss.item() - total) <= 1e-5 * total
    assert (g - gradient(m, images)).abs().max().item() <= BOUND


def test_batched_step():
    cameras, _, m, images = problem()
    batch = hsgd.Batch(1, 1, N, H, W, 1, dtype=torch.float32)
    st = hsgd.ServingStream(0, *cameras, W, H, (1,), 1, dtype=torch.float32,
                            lr_rgb=0.25, lr_alpha=0.25)
    st.levels[0].copy_(m)
    st.images[0].copy_(images)
    assert batch.admit(st) is not None
    assert batch.step()[0] == 1
    want = (m - 0.25 * gradient(m, images)).clamp_(0.0, 1.0)
    assert (st.result - want).abs().max().item() <= BOUND
    total = squares(m, images)
    assert abs(st.loss_log[0].item() - total) <= 1e-5 * total


def test_translation_gradient():
    _, table, m, images = problem()
    assert table.shift_only
    g, loss = hsgd.hsgd_grad_step(m, table, N, images=images, want_grad=True, want_loss=True)
    total = squares(m, images)
    assert abs(loss.item() - total) <= 1e-5 * total
    assert (g - gradient(m, images)).abs().max().item() <= BOUND


@pytest.mark.parametrize("general", [False, True], ids=["translation", "general"])
@pytest.mark.parametrize("n,h", [(1, 5 << 20), (3, 3 << 19)], ids=["planes", "views"])
def test_plane_sweep(n, h, general):
    """More planes of one view than a launch holds, and more views."""
    D = 64
    eye = np.eye(3)
    table = hsgd.psv_warps(eye, np.stack([eye] * n), np.stack([eye] * n), np.zeros((n, 3)), np.linspace(1.0, 2.0, D))
    images = torch.rand((n, h, W, 3), device="cuda")
    out, = hsgd.hsgd_plane_sweep(images, table.tensor if general else table, D, dtype=torch.bfloat16)
    for view, image in zip(out, images.to(torch.bfloat16)):
        assert all(torch.equal(plane, image) for plane in view)


def test_conversion():
    src = torch.rand((1 << 32) + 4097, device="cuda")
    assert torch.equal(hsgd.hsgd_convert(src, torch.bfloat16), src.to(torch.bfloat16))
