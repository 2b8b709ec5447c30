"""The first kernel of a batched step: selection, upsampling fused with selection and target
pyramids of different requests in one launch. Requests of the smallest frames, of widths
around its 62-column blocks and of every level count, together in one batch and out of phase,
each equal (bitwise) to the same refinement on its own, which uses other kernels for all three.
"""

import pytest
import torch

from paper_2307_03017_amd import hsgd
from tests._problems import rig

pytestmark = pytest.mark.gpu

# (W, H, D of 8, iterations per level, rule); D scales with the batch's plane count
FRAMES = [
    (4, 4, 8, (1, 1), "topk"),                # a coarsest level of 2 x 2
    (248, 16, 5, (1, 1), "topk"),             # 124 columns: two blocks exactly
    (252, 12, 8, (2, 1), "mvs"),              # 126: a third block of two columns
    (132, 36, 3, (0, 1, 1), "topk"),          # upsampling and pyramid in the same step
    (136, 24, 7, (1, 1, 1, 1), "topk"),   # three levels below
    (50, 34, 6, (2,), "topk"),                # no levels below
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("planes", [8, 16, 24, 32, 40, 48, 64])
def test_mixed_requests_equal_refine(planes, dtype):
    N, k = 2, 2
    gen = torch.Generator(device="cuda").manual_seed(planes)
    batch = hsgd.Batch(len(FRAMES), planes, N, 36, 252, k, dtype=dtype)
    streams, alone = [], []
    for i, (W, H, d, iters, rule) in enumerate(FRAMES):
        D, L = d * planes // 8, len(iters)
        rg = rig(i, N, D, W, H, 0.8 * W, 0.1)
        args = [rg[a] for a in ("K_ref", "K", "R", "t", "depths")]
        images = torch.rand((N, H, W, 3), generator=gen, device="cuda")
        init = torch.rand((D, H >> (L - 1), W >> (L - 1), 4), generator=gen, device="cuda").to(dtype)
        st = hsgd.ServingStream(i, *args, W, H, iters, k, dtype=dtype, lr_rgb=0.5, lr_alpha=0.5, rule=rule)
        st.levels[0].copy_(init)
        st.images[-1].copy_(images)
        streams.append(st)
        alone.append(hsgd.hsgd_refine(init, images, *args, iters, k, lr_rgb=0.5, lr_alpha=0.5, rule=rule))
    torch.cuda.synchronize()
    for i, st in enumerate(streams):          # one more request from each step on
        assert batch.admit(st) is not None
        if i % 2:
            batch.step()
    while batch.step()[0]:
        pass
    torch.cuda.synchronize()
    for st, (want, losses) in zip(streams, alone):
        assert torch.equal(st.result, want)
        assert torch.equal(st.loss_log[:sum(st.iters)], losses)
