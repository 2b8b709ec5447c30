"""The calls whose speed this framework is held to, over the sizes that its users have.

Every case names a kind of call and its sizes; `prepare` makes what a program has in hand
before the call (inputs on the GPU, camera tables, plans, streams), `run` is the call itself
through the package's public entry points, `exact` the same result in 64 bits from plain
torch. Cameras are forward facing: N views shifted by up to a in x and y around the
reference, `tilt` radians of rotation and +-2 tilt along z where they are hand held; planes
are uniform in inverse depth from 1 to 100. Scenes are piecewise constant textures on one
surface per pixel; an MPI that is being refined is that surface with noise on its alpha
logits (sigma 0.5) and colours (sigma 0.1).
"""

from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2307_03017_amd import autograd, hsgd

DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}


def _refine(W, H, D, N, k, iters, dtype="fp32", a=0.1, prior=0.0):
    return {"kind": "refine", "W": W, "H": H, "D": D, "N": N, "k": k, "iters": iters, "dtype": dtype, "a": a,
            "prior": prior, "tilt": 0.0}


def _case(kind, W, H, D, N, dtype="fp32", tilt=0.0, a=0.1, **more):
    return {"kind": kind, "W": W, "H": H, "D": D, "N": N, "dtype": dtype, "a": a, "tilt": tilt, **more}


def listed():
    return [
        # the tiny frame of the smoke check and of a C program's first call: launches count
        dict(_refine(64, 48, 8, 3, 2, "2,1", a=0.05), name="refine 64x48x8"),
        # the benchmark frame
        dict(_refine(512, 384, 32, 4, 4, "1,1,1"), name="refine 512x384x32"),
        # the paper's frame: 40 planes, five kept, three iterations, with the sparsity prior
        dict(_refine(512, 378, 40, 3, 5, "1,2", prior=100.0), name="refine 512x378x40"),
        # the large XR frame
        dict(_refine(1920, 1080, 64, 8, 3, "0,1,1,1", "bf16", a=0.15), name="refine 1920x1080x64 bf16"),
        # one descent step of a program's own loop, hand-held cameras (general homographies)
        dict(_case("step", 512, 384, 32, 4, tilt=0.01, k=4), name="step 512x384x32 tilted"),
        # continuous batching: one frame of each of eight resident scenes
        {"name": "serve 8 scenes bf16", "kind": "serve", "dtype": "bf16", "a": 0.1, "tilt": 0.0,
         "scenes": "256x192x16x3x2 256x192x16x4x2 256x192x16x5x2 512x384x32x3x4 512x384x32x4x4 512x384x32x5x4 "
                   "1008x756x32x3x4 1008x756x32x5x4"},
        # the 18 views of a light-field display from a finished MPI
        dict(_case("render", 512, 384, 32, 18), name="render 18 of 512x384x32"),
        # one frame of a viewer whose camera turns
        dict(_case("render", 1008, 756, 32, 1, "bf16", tilt=0.01), name="render 1008x756x32 bf16 tilted"),
        # dense gradient of the photometric loss through autograd (an optimiser's step)
        dict(_case("loss", 256, 192, 16, 3), name="loss backward 256x192x16"),
        # rendering inside somebody's own loss: forward, then the adjoint of an image gradient
        dict(_case("vjp", 501, 333, 24, 2, tilt=0.01), name="render vjp 501x333x24 tilted"),
        # the plane-sweep volume that feeds the initial MPI
        dict(_case("sweep", 512, 384, 32, 4, levels=3), name="sweep 512x384x32"),
        # the same for hand-held captures, 16-bit volume
        dict(_case("sweep", 1008, 756, 32, 5, "bf16", tilt=0.01, levels=3), name="sweep 1008x756x32 bf16 tilted"),
    ]


def draw(rng):
    """Sizes spread over their logarithm from 64x48 to the large frames, odd ones among them."""
    kind = rng.choice(["refine", "refine", "refine", "step", "serve", "render", "render", "loss", "vjp", "sweep", "sweep"])
    dtype = rng.choice(["fp32", "fp32", "bf16"])

    def frame(most_w, m):
        w = math.exp(rng.uniform(math.log(64), math.log(most_w)))
        return max(1, round(w / m)) * m, max(1, round(w * rng.uniform(0.55, 0.8) / m)) * m

    def planes(most):
        return rng.choice([8, 16, 32, most, round(math.exp(rng.uniform(math.log(4), math.log(most))))])

    tilt = rng.choice([0.0, 0.005, 0.01])
    if kind == "refine":
        its = rng.choice(["1,1,1", "1,2", "2,1", "0,1,1,1", "1,1", "3"])
        W, H = frame(1280, 1 << its.count(","))
        D = planes(64)
        return _refine(W, H, D, rng.randint(2, 6), min(D, rng.randint(2, 5)), its, dtype, rng.choice([0.05, 0.1, 0.15]),
                       rng.choice([0.0, 0.0, 100.0]))
    if kind == "serve":
        some = []
        for _ in range(rng.randint(2, 8)):
            W, H = frame(1024, 4)
            some.append("%dx%dx%dx%dx%d" % (W, H, rng.choice([8, 16, 24, 32]), rng.randint(3, 5), rng.randint(2, 4)))
        return {"kind": "serve", "dtype": dtype, "a": 0.1, "tilt": 0.0, "scenes": " ".join(some)}
    if kind == "sweep":
        levels = rng.randint(1, 4)
        W, H = frame(1024, 1 << (levels - 1))
        return _case("sweep", W, H, planes(40), rng.randint(2, 5), dtype, rng.choice([0.0, 0.0, tilt]), levels=levels)
    if kind == "render":
        W, H = frame(1440, 1)
        return _case("render", W, H, planes(64), rng.choice([1, 2, 5, 18]), dtype, tilt)
    W, H = frame(1024 if kind == "step" else 640, 1)
    D = planes(48)
    more = {"k": min(D, rng.randint(2, 5))} if kind == "step" else {}
    return _case(kind, W, H, D, rng.randint(2, 5), "fp32" if kind == "loss" else dtype, tilt, **more)


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _depths(D):
    return 1.0 / (1.0 - np.arange(D) * 0.99 / max(D - 1, 1))


def _cameras(c, seed):
    """K_ref [3][3], K [N][3][3], R [N][3][3], t [N][3], depths [D]: world to camera."""
    r = np.random.default_rng([seed, 1])
    W, H, N = c["W"], c["H"], c["N"]
    K = np.array([[0.78125 * W, 0.0, (W - 1) / 2.0], [0.0, 0.78125 * W, (H - 1) / 2.0], [0.0, 0.0, 1.0]])
    t = np.concatenate([r.uniform(-c["a"], c["a"], (N, 2)), np.zeros((N, 1))], axis=1)
    R = np.repeat(np.eye(3)[None], N, axis=0)
    if c["tilt"]:
        for i, (x, y, z) in enumerate(r.normal(0.0, c["tilt"], (N, 3))):
            X = np.array([[1, 0, 0], [0, math.cos(x), -math.sin(x)], [0, math.sin(x), math.cos(x)]])
            Y = np.array([[math.cos(y), 0, math.sin(y)], [0, 1, 0], [-math.sin(y), 0, math.cos(y)]])
            Z = np.array([[math.cos(z), -math.sin(z), 0], [math.sin(z), math.cos(z), 0], [0, 0, 1]])
            R[i] = Z @ Y @ X
        t[:, 2] = r.uniform(-2 * c["tilt"], 2 * c["tilt"], N)
    return K, np.repeat(K[None], N, axis=0), R, t, _depths(c["D"])


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 11)


def _surface(c, seed, w, h):
    """The scene's MPI at w x h: [D][h][w][4] float32, alpha 1 on the plane nearest to a smooth
    field of inverse depths and 0 elsewhere, per plane a grid of random colours."""
    g, D = _generator(seed), c["D"]
    field = torch.rand((1, 1, 5, 6), generator=g, device="cuda") * 0.99 + 0.01
    cells = torch.rand((D, 9, 13, 3), generator=g, device="cuda")
    u = ((torch.arange(w, device="cuda") + 0.5) / w)
    v = ((torch.arange(h, device="cuda") + 0.5) / h)
    at = torch.stack(torch.broadcast_tensors((2 * u - 1)[None, :], (2 * v - 1)[:, None]), dim=-1)[None]
    inverse = F.grid_sample(field, at, align_corners=True, padding_mode="border")[0, 0]
    plane = ((1.0 - inverse) * (max(D - 1, 1) / 0.99)).round().clamp(0, D - 1).long()
    m = torch.empty((D, h, w, 4), device="cuda")
    m[..., :3] = cells[:, (v * 9).long()][:, :, (u * 13).long()]
    m[..., 3] = plane[None] == torch.arange(D, device="cuda")[:, None, None]
    return m


def _state(c, seed, w, h):
    """An MPI as a refinement meets it: the surface with noise, in the case's storage."""
    m = _surface(c, seed, w, h)
    g = _generator(seed + 1_000_003)
    logit = torch.logit(m[..., 3].clamp(0.01, 0.99))
    logit += 0.5 * torch.randn(logit.shape, generator=g, device="cuda")
    m[..., 3] = torch.sigmoid(logit)
    for ch in range(3):
        m[..., ch] = (m[..., ch] + 0.1 * torch.randn(logit.shape, generator=g, device="cuda")).clamp_(0.0, 1.0)
    return m.to(DTYPES[c["dtype"]])


def _targets(c, seed):
    """What the N cameras see of the scene: [N][H][W][3] float32."""
    W, H = c["W"], c["H"]
    maps = _view_maps(_cameras(c, seed), W, H, W, H)
    m = _surface(c, seed, W, H).reshape(c["D"], H * W, 4)
    return torch.stack([_composite(m, one, H, W)[0] for one in maps]).reshape(c["N"], H, W, 3).contiguous()


def _noise_like(shape, seed):
    return torch.randn(shape, generator=_generator(seed + 2_000_003), device="cuda")


def _levels(c):
    its = [int(i) for i in c["iters"].split(",")]
    L = len(its)
    return its, [(c["W"] >> (L - 1 - l), c["H"] >> (L - 1 - l)) for l in range(L)]


def _scenes(c):
    out = []
    for i, s in enumerate(c["scenes"].split()):
        W, H, D, N, k = (int(x) for x in s.split("x"))
        out.append(_refine(W, H, D, N, k, "1,1,1", c["dtype"], c["a"]))
    return out


def _table(c, seed):
    W, H = c["W"], c["H"]
    return hsgd.level_warps(*_cameras(c, seed), W, H, W, H)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "refine":
        its, shapes = _levels(c)
        plan = hsgd.RefinePlan(*_cameras(c, seed), c["W"], c["H"], its, c["k"], dtype=DTYPES[c["dtype"]],
                               lambda_s=c["prior"])
        images = _targets(c, seed)
        return {"kind": kind, "plan": plan, "images": images, "init": _state(c, seed, *shapes[0]),
                "descriptors": plan.descriptors(images)}
    if kind == "serve":
        scenes = _scenes(c)
        most = {f: max(s[f] for s in scenes) for f in ("D", "N", "H", "W", "k")}
        batch = hsgd.Batch(max(8, len(scenes)), most["D"], most["N"], most["H"], most["W"], most["k"],
                           dtype=DTYPES[c["dtype"]], hbm_budget=1 << 36)
        streams, inits = [], []
        for i, s in enumerate(scenes):
            its, shapes = _levels(s)
            st = hsgd.ServingStream(i, *_cameras(s, seed + 31 * i), s["W"], s["H"], its, s["k"], dtype=DTYPES[c["dtype"]])
            st.images[-1].copy_(_targets(s, seed + 31 * i))
            streams.append(st)
            inits.append(_state(s, seed + 31 * i, *shapes[0]))
        return {"kind": kind, "batch": batch, "streams": streams, "inits": inits}
    if kind == "sweep":
        dtype = DTYPES[c["dtype"]]
        out = [torch.empty((c["N"], c["D"], c["H"] >> l, c["W"] >> l, 3), dtype=dtype, device="cuda")
               for l in range(c["levels"])]
        return {"kind": kind, "images": _targets(c, seed), "table": hsgd.psv_warps(*_cameras(c, seed)), "D": c["D"],
                "levels": c["levels"], "dtype": dtype, "out": out}
    state = {"kind": kind, "table": _table(c, seed), "N": c["N"], "mpi": _state(c, seed, c["W"], c["H"])}
    if kind == "step":
        state.update(images=_targets(c, seed), k=c["k"], work=torch.empty_like(state["mpi"]))
        state["ws"] = hsgd.workspace(hsgd.OP_GRAD_STEP, c["D"], c["H"], c["W"], c["N"], c["k"])
    elif kind == "loss":
        state.update(images=_targets(c, seed), master=state["mpi"].requires_grad_())
    elif kind == "vjp":
        state.update(master=state["mpi"].float().requires_grad_(),
                     upstream=_noise_like((c["N"], c["H"], c["W"], 3), seed) * 0.1)
    return state


def run(state):
    s, kind = state, state["kind"]
    if kind == "refine":
        plan = s["plan"]
        plan.levels[0].copy_(s["init"])
        return {"mpi": plan.run(s["images"], s["descriptors"]), "loss": plan.loss_log}
    if kind == "serve":
        for st, init in zip(s["streams"], s["inits"]):
            if s["batch"].admit(st) is None:
                raise RuntimeError("a frame was refused")
            st.levels[0].copy_(init)
        while s["batch"].step()[0]:
            pass
        return [{"mpi": st.result, "loss": st.loss_log} for st in s["streams"]]
    if kind == "step":
        m = s["work"].copy_(s["mpi"])          # the step works in place
        mask = hsgd.hsgd_select_active(m, s["k"], with_ids=False)
        _, loss = hsgd.hsgd_grad_step(m, s["table"], s["N"], images=s["images"], mask=mask, kcap=s["k"], lr_rgb=1.0,
                                      lr_alpha=1.0, want_loss=True, ws=s["ws"])
        return {"mpi": m, "mask": mask, "loss": loss}
    if kind == "render":
        return hsgd.hsgd_render(s["mpi"], s["table"], s["N"])[0]
    if kind == "loss":
        loss = autograd.photometric_loss(s["master"], s["table"], s["images"])
        return {"loss": loss, "grad": torch.autograd.grad(loss, s["master"])[0]}
    if kind == "vjp":
        storage = None if s["mpi"].dtype == torch.float32 else s["mpi"]
        out = autograd.render(s["master"], s["table"], s["N"], storage=storage)
        return {"views": out, "grad": torch.autograd.grad(out, s["master"], s["upstream"])[0]}
    return hsgd.hsgd_plane_sweep(s["images"], s["table"], s["D"], s["levels"], out=s["out"], dtype=s["dtype"])


# ---------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------
def work(case):
    """Inputs read once, outputs written once. Operations: 37 per sample of a view (bilinear
    RGBA 28, over 9) and 21 more for its adjoint, 32 per selected voxel and view for the
    transposed bilinear; 21 per sample of a plane-sweep volume and 4 per pooled value."""
    c, kind = case, case["kind"]
    if kind == "serve":
        all_ = [work(s) for s in _scenes(c)]
        return {"bytes": sum(w["bytes"] for w in all_), "flops": sum(w["flops"] for w in all_)}
    W, H, D, N = c["W"], c["H"], c["D"], c["N"]
    HW, s = W * H, 16 if c["dtype"] == "fp32" else 8
    if kind == "refine":
        its, shapes = _levels(c)
        w0, h0 = shapes[0]
        steps = sum(n * w * h for n, (w, h) in zip(its, shapes))
        return {"bytes": D * w0 * h0 * s + N * HW * 12 + D * HW * s, "flops": N * steps * (58 * D + 32 * c["k"])}
    if kind == "step":
        return {"bytes": 2 * D * HW * s + N * HW * 12 + 8 * HW, "flops": N * HW * (58 * D + 32 * c["k"])}
    if kind == "render":
        return {"bytes": D * HW * s + N * HW * 12, "flops": N * HW * 37 * D}
    if kind == "loss":
        return {"bytes": D * HW * (s + 16) + N * HW * 12, "flops": N * HW * (58 + 32) * D}
    if kind == "vjp":
        return {"bytes": D * HW * (s + 16) + 2 * N * HW * 12, "flops": N * HW * (58 + 32 + 37) * D}
    one = 3 * (4 if c["dtype"] == "fp32" else 2)
    samples = sum(N * D * (H >> l) * (W >> l) for l in range(c["levels"]))
    return {"bytes": N * HW * 12 + samples * one, "flops": N * D * HW * 21 + (samples - N * D * HW) * 12}


# ---------------------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------
def _plane_maps(cameras, W, H, w, h):
    """Reference pixel -> view pixel on each plane, for a w x h level of a W x H rig: [N][D][3][3]."""
    Kr, K, R, t, depths = cameras

    def scaled(k):
        k = k.copy()
        k[0] *= w / W
        k[1] *= h / H
        k[0, 2] += 0.5 * w / W - 0.5
        k[1, 2] += 0.5 * h / H - 0.5
        return k

    back = np.linalg.inv(scaled(Kr))
    n = np.array([0.0, 0.0, 1.0])
    return [[scaled(K[i]) @ (R[i] + np.outer(t[i], n) / d) @ back for d in depths] for i in range(len(K))]


def _view_maps(cameras, W, H, w, h):
    """View pixel -> reference pixel on each plane."""
    return [[np.linalg.inv(m) for m in one] for one in _plane_maps(cameras, W, H, w, h)]


def _taps(G, H, W, dtype):
    """The four bilinear taps of every pixel under the map G: [(flat index, weight)], weight 0
    outside the plane and behind the camera."""
    y, x = torch.meshgrid(torch.arange(H, device="cuda", dtype=torch.float64),
                          torch.arange(W, device="cuda", dtype=torch.float64), indexing="ij")
    x, y = x.reshape(-1), y.reshape(-1)
    q = [float(G[r][0]) * x + float(G[r][1]) * y + float(G[r][2]) for r in range(3)]
    front = q[2] > 0
    z = torch.where(front, q[2], torch.ones_like(q[2]))
    u, v = (q[0] / z).clamp(-4.0, W + 4.0), (q[1] / z).clamp(-4.0, H + 4.0)
    x0, y0 = u.floor(), v.floor()
    fx, fy = u - x0, v - y0
    x0, y0 = x0.long(), y0.long()
    out = []
    for dx, dy, wt in ((0, 0, (1 - fx) * (1 - fy)), (1, 0, fx * (1 - fy)), (0, 1, (1 - fx) * fy), (1, 1, fx * fy)):
        xx, yy = x0 + dx, y0 + dy
        ok = front & (xx >= 0) & (xx < W) & (yy >= 0) & (yy < H)
        out.append((yy.clamp(0, H - 1) * W + xx.clamp(0, W - 1), torch.where(ok, wt, torch.zeros_like(wt)).to(dtype)[:, None]))
    return out


def _sample(plane, taps):
    return sum(plane[i] * w for i, w in taps)


def _composite(m, maps, H, W, keep=False):
    """One view of m [D][H W][4]: (colour [H W][3], the transmittance before each plane)."""
    T = torch.ones(H * W, 1, device="cuda", dtype=m.dtype)
    C = torch.zeros(H * W, 3, device="cuda", dtype=m.dtype)
    before = []
    for z, G in enumerate(maps):
        s = _sample(m[z], _taps(G, H, W, m.dtype))
        if keep:
            before.append(T)
        C = C + T * s[:, 3:] * s[:, :3]
        T = T * (1.0 - s[:, 3:])
    return C, before


def _adjoint(m, maps, H, W, before, g, grad):
    """Adds the gradient of one view with upstream g [H W][3] to grad [D][H W][4]."""
    B = torch.zeros_like(g)
    for z in range(len(maps) - 1, -1, -1):
        taps = _taps(maps[z], H, W, m.dtype)
        s = _sample(m[z], taps)
        c, a = s[:, :3], s[:, 3:]
        gs = torch.cat([g * a * before[z], before[z] * (g * (c - B)).sum(1, keepdim=True)], dim=1)
        B = a * c + (1.0 - a) * B
        for i, w in taps:
            grad[z].index_add_(0, i, gs * w)


def _gradient(m, views, H, W, images):
    """(photometric loss, its dense gradient) of m [D][H W][4]."""
    N, grad, loss = len(views), torch.zeros_like(m), 0.0
    for maps, image in zip(views, images):
        C, before = _composite(m, maps, H, W, keep=True)
        r = C - image.reshape(-1, 3).double()
        loss = loss + (r * r).sum() / (2 * N)
        _adjoint(m, maps, H, W, before, r / N, grad)
    return loss, grad


def _selected(alpha, k):
    """The k planes of largest a T per pixel as booleans [D][H W]; scores are 32-bit by contract."""
    a = alpha.float()
    T, A = torch.ones_like(a[0]), torch.empty_like(a)
    for z in range(len(a)):
        A[z] = a[z] * T
        T = T * (1.0 - a[z])
    kept = torch.zeros(a.shape, dtype=torch.bool, device=a.device)
    for _ in range(min(k, len(a))):
        best, top = torch.full_like(A[0], -2.0), torch.zeros(A[0].shape, dtype=torch.long, device=a.device)
        for z in range(len(a)):
            more = ~kept[z] & (A[z] > best)
            best, top = torch.where(more, A[z], best), torch.where(more, torch.full_like(top, z), top)
        kept.scatter_(0, top[None], True)
    return kept


def _stored(m, dtype):
    return m.to(torch.bfloat16).double() if dtype == "bf16" else m


def _descend(m, views, H, W, images, k, prior, dtype):
    kept = _selected(m[..., 3], k)
    loss, g = _gradient(m, views, H, W, images)
    if prior:
        d = 0.5 - m[..., 3]
        g[..., 3] += prior * torch.sign(d) / (1.5 - d.abs()) / d.numel()
    new = _stored((m - g).clamp(0.0, 1.0), dtype)
    return torch.where(kept[..., None], new, m), loss, kept


def _refined(c, seed):
    its, shapes = _levels(c)
    W, H, D = c["W"], c["H"], c["D"]
    cameras, losses = _cameras(c, seed), []
    images = [_targets(c, seed).double()]
    for _ in shapes[1:]:
        images.insert(0, F.avg_pool2d(images[0].permute(0, 3, 1, 2), 2).permute(0, 2, 3, 1))
    m = _state(c, seed, *shapes[0]).double()
    for l, (w, h) in enumerate(shapes):
        if l:
            up = F.interpolate(m.permute(0, 3, 1, 2), scale_factor=2, mode="bilinear", align_corners=False)
            m = _stored(up.permute(0, 2, 3, 1).contiguous(), c["dtype"])
        m = m.reshape(D, h * w, 4)
        for _ in range(its[l]):
            m, loss, _ = _descend(m, _view_maps(cameras, W, H, w, h), h, w, images[l], c["k"], c["prior"], c["dtype"])
            losses.append(loss)
        m = m.reshape(D, h, w, 4)
    return {"mpi": m, "loss": torch.stack(losses)}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "refine":
        return _refined(c, seed)
    if kind == "serve":
        return [_refined(s, seed + 31 * i) for i, s in enumerate(_scenes(c))]
    W, H, D = c["W"], c["H"], c["D"]
    cameras = _cameras(c, seed)
    if kind == "sweep":
        images = _targets(c, seed).double().reshape(c["N"], H * W, 3)
        out = [torch.stack([torch.stack([_sample(images[i], _taps(G, H, W, torch.float64)) for G in one])
                            for i, one in enumerate(_plane_maps(cameras, W, H, W, H))]).reshape(c["N"], D, H, W, 3)]
        for l in range(1, c["levels"]):
            p = out[-1]
            out.append(0.25 * (p[:, :, ::2, ::2] + p[:, :, 1::2, ::2] + p[:, :, ::2, 1::2] + p[:, :, 1::2, 1::2]))
        return out
    views = _view_maps(cameras, W, H, W, H)
    m = _state(c, seed, W, H).double().reshape(D, H * W, 4)
    if kind == "render":
        return torch.stack([_composite(m, one, H, W)[0] for one in views]).reshape(-1, H, W, 3)
    if kind == "step":
        new, loss, _ = _descend(m, views, H, W, _targets(c, seed), c["k"], 0.0, c["dtype"])
        return {"mpi": new.reshape(D, H, W, 4), "mask": None, "loss": loss.reshape(1)}
    if kind == "loss":
        loss, grad = _gradient(m, views, H, W, _targets(c, seed))
        return {"loss": loss, "grad": grad.reshape(D, H, W, 4)}
    grad, out = torch.zeros_like(m), []
    upstream = (_noise_like((c["N"], H, W, 3), seed) * 0.1).double().reshape(c["N"], H * W, 3)
    for maps, g in zip(views, upstream):
        C, before = _composite(m, maps, H, W, keep=True)
        out.append(C.reshape(H, W, 3))
        _adjoint(m, maps, H, W, before, g, grad)
    return {"views": torch.stack(out), "grad": grad.reshape(D, H, W, 4)}
