"""Performance cases: what a user of the splatting library has it do, through its public entry points.

A case is one of these kinds:
  step     a training step: differentiable render of a Gaussian set, then its backward to every parameter
  render   a frame without gradients (evaluation, novel views)
  distil   the learned colour decoder's fused forward, loss and backward on a batch of directions
  update   what follows the raster in a training iteration: the L1 loss of an image and one Adam step
  density  one round of density control
The scenes follow the library's workloads: uniform Gaussians, or clusters with a 100x density skew, isotropic or
stretched up to 20:1.  Everything is drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_2510_14564_amd import gs, scenes
from paper_2510_14564_amd.decoder import Decoder
from paper_2510_14564_amd.raster import Rasterizer, l1_loss, rasterize, rasterize_learned

DEV = "cuda"
PARAMS = ("means", "log_scales", "quats", "logits", "sh")
LRS = dict(means=1.6e-4, log_scales=5e-3, quats=1e-3, logits=5e-2, sh_dc=2.5e-3, sh_rest=1.25e-4)
# the compositing's work per pixel, as the library's workloads have it: pairs walked and blended
WALKED, BLENDED = 200.0, 32.0


def _step(name, n, width, height, degree, scene="skewed", view="orbit", **more):
    c = dict(name=name, kind="step", n=n, width=width, height=height, degree=degree, scene=scene, view=view,
             learned=False, deterministic=False, hashed=False, no_wait=False)
    c.update(more)
    return c


def listed():
    return [
        # a toy scene, as in unit tests, demos and the first steps of a run: launches and host time count
        _step("step_tiny", 4096, 128, 128, 0, scene="uniform", view="front"),
        # a mid-size scene at a square resolution, the usual settings
        _step("step_skewed", 200_000, 800, 800, 3, view="front"),
        # the flagship training step, queued without waiting for the list length
        _step("step_main", 1_000_000, 1600, 1064, 3, no_wait=True),
        # the largest: many long, stretched Gaussians, the longest tile lists
        _step("step_heavy", 1_500_000, 1920, 1080, 3, scene="stretched"),
        # colour from the learned decoder in place of spherical harmonics
        _step("step_learned", 200_000, 800, 800, 3, view="front", learned=True),
        # reproducible gradients, at a size and degree that fill no tile evenly
        _step("step_deterministic", 120_001, 1237, 823, 2, deterministic=True),
        # the approximate colour-hash sampling mode
        _step("step_hashed", 200_000, 800, 800, 3, view="front", hashed=True),
        # evaluation of a trained set at 4K
        dict(name="render_uhd", kind="render", n=1_000_000, width=3840, height=2160, degree=3, scene="skewed",
             view="orbit"),
        # a thumbnail of a large set, of odd size: few tiles, each with a long list
        dict(name="render_thumbnail", kind="render", n=500_001, width=203, height=131, degree=1, scene="skewed",
             view="orbit"),
        # one minibatch of decoder distillation: 16,384 Gaussians, 64 directions each
        dict(name="distil", kind="distil", n=16_384, per=64),
        # the rest of the flagship training iteration
        dict(name="update_main", kind="update", n=1_000_000, width=1600, height=1064, degree=3),
        # density control between training intervals
        dict(name="density_skewed", kind="density", n=200_000, radius=0.03),
    ]


def draw(rng):
    def lu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(("step", "render", "distil", "update", "density"), (8, 3, 1, 1, 1))[0]
    if kind == "distil":
        per = rng.choice((1, 4, 16, 64))
        return dict(kind=kind, n=lu(64, 20_000) * (64 // per) // 4, per=per)
    if kind == "density":
        n = lu(5_000, 600_000)
        return dict(kind=kind, n=n, radius=round(0.03 * (200_000 / n) ** (1 / 3), 5))  # about 20 neighbours
    width, height = lu(96, 3840), lu(96, 2160)
    degree = rng.choice((0, 1, 2, 3, 3))
    if kind == "update":
        return dict(kind=kind, n=lu(1_000, 2_000_000), width=width, height=height, degree=degree)
    scene = rng.choice(("uniform", "skewed", "skewed", "stretched"))
    most = {"uniform": 1.5e11, "skewed": 3e12, "stretched": 1.5e12}[scene] / (width * height)
    n = min(lu(2_000, 1_500_000), int(most), 1_500_000)
    view = rng.choice(("front", "orbit"))
    if kind == "render":
        return dict(kind=kind, n=n, width=width, height=height, degree=degree, scene=scene, view=view)
    option = rng.choice(("none", "none", "none", "learned", "deterministic", "hashed", "no_wait"))
    c = _step("", n, width, height, degree, scene=scene, view=view)
    if option != "none" and not (option == "no_wait" and width * height > 4_000_000):
        c[option] = True
    if option == "deterministic":
        c["n"] = min(n, 200_000, int(4e11 / (width * height)))  # a row of partial sums per list entry
    del c["name"]
    return c


# --------------------------------------------------------------------- inputs


def _rand(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape, std=1.0, mean=0.0):
    return torch.randn(shape, generator=g, device=DEV) * std + mean


def _uniform(g, *shape, lo=0.0, hi=1.0):
    return torch.rand(shape, generator=g, device=DEV) * (hi - lo) + lo


def _scene(g, n, degree, kind):
    """Parameter arrays of n Gaussians, with the distributions of the library's workloads."""
    if kind == "uniform":
        means = _uniform(g, 3, n, lo=-1.0, hi=1.0)
        log_scales = _normal(g, 3, n, std=0.5, mean=-3.5)
    else:
        count = 256 if kind == "stretched" else 64
        w = 100.0 ** (torch.arange(count, device=DEV) / (count - 1))
        centres = _uniform(g, 3, count, lo=-1.0, hi=1.0)
        label = torch.multinomial(w / w.sum(), n, replacement=True, generator=g)
        means = centres[:, label] + _normal(g, 3, n, std=0.1)
        if kind == "stretched":
            base = _normal(g, n, std=0.7, mean=-4.5)
            ratio = math.log(20.0) * _uniform(g, n)
            axis = torch.randint(0, 3, (n,), generator=g, device=DEV)
            log_scales = (base - ratio / 3.0).repeat(3, 1)
            log_scales[axis, torch.arange(n, device=DEV)] += ratio
        else:
            log_scales = _normal(g, 3, n, std=0.7, mean=-4.5)
    quats = _normal(g, 4, n)
    quats /= quats.norm(dim=0, keepdim=True)
    nc = (degree + 1) ** 2
    sh = _normal(g, nc, 3, n, std=0.05)
    sh[0] *= 6.0 if kind == "uniform" else 10.0
    return dict(means=means.contiguous(), log_scales=log_scales.contiguous(), quats=quats,
                logits=_normal(g, n), sh=sh)


def _camera(case, seed):
    if case["view"] == "front":
        return scenes.front_camera(case["width"], case["height"])
    return scenes.orbit_camera(int(seed) % 32, 32, case["width"], case["height"])


def _bf16(x):
    """Values rounded to bfloat16, and their bit patterns."""
    b = x.to(torch.bfloat16)
    return b.float(), b.view(torch.int16)


def _decoder_inputs(g, n):
    """BF16 latents [n][16] and Kaiming weights with zero biases, in the library's order."""
    z = _bf16(_normal(g, n, 16, std=0.1))
    parts = []
    for rows, cols in ((64, 32), (64, 64), (3, 64)):
        b = math.sqrt(6.0 / cols)
        parts += [_uniform(g, rows * cols, lo=-b, hi=b), torch.zeros(rows, device=DEV)]
    return z, _bf16(torch.cat(parts))


def _frame_inputs(case, seed):
    g = _rand(seed)
    p = _scene(g, case["n"], case["degree"], case["scene"])
    G = _normal(g, 3, case["height"], case["width"])
    dec = _decoder_inputs(g, case["n"]) if case.get("learned") else None
    return p, G, dec


def _distil_inputs(case, seed):
    g = _rand(seed)
    z, w = _decoder_inputs(g, case["n"])
    d = _normal(g, case["n"] * case["per"], 3)
    d /= d.norm(dim=1, keepdim=True)
    return z, w, d, _uniform(g, case["n"] * case["per"], 3)


def _update_inputs(case, seed):
    g = _rand(seed)
    p = _scene(g, case["n"], case["degree"], "skewed")
    grads = {k: _normal(g, *v.shape, std=1e-4) for k, v in p.items()}
    m = {k: _normal(g, *v.shape, std=1e-4) for k, v in p.items()}
    v2 = {k: _normal(g, *v.shape, std=1e-4).square() for k, v in p.items()}
    img = _uniform(g, 3, case["height"], case["width"])
    return p, grads, m, v2, img, _uniform(g, 3, case["height"], case["width"])


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "render"):
        p, G, dec = _frame_inputs(case, seed)
        schedule = gs.SCHEDULE_BALANCED | (gs.RENDER_COLOUR_HASH if case.get("hashed") else 0)
        rast = Rasterizer(_camera(case, seed), case["degree"], deterministic=bool(case.get("deterministic")),
                          schedule=schedule, async_k=bool(case.get("no_wait")))
        st = dict(kind=kind, p=p, rast=rast)
        if kind == "step":
            st["G"] = G
            leaves = [p[k] for k in PARAMS[:4]]
            if dec is not None:
                (_, zb), (_, wb) = dec
                d = Decoder(case["n"], latents_bits=zb.cpu().numpy().view("uint16"),
                            params_bits=wb.cpu().numpy().view("uint16"))
                d.latents.requires_grad_(True)
                d.params.requires_grad_(True)
                st["dec"] = d
                leaves += [d.latents, d.params]
            else:
                leaves.append(p["sh"])
            st["leaves"] = [t.requires_grad_(True) for t in leaves]
        return st
    if kind == "distil":
        (_, zb), (_, wb), dirs, target = _distil_inputs(case, seed)
        S = case["n"] * case["per"]
        packed = torch.empty(gs.MLP_PACKED_BYTES // 4 + 4, dtype=torch.float32, device=DEV)
        gs.mlp_pack(wb, packed)
        return dict(kind=kind, S=S, per=case["per"], z=zb, dirs=dirs, target=target, packed=packed,
                    dlat=torch.empty((case["n"], 16), device=DEV), dw=torch.empty(gs.MLP_PARAMS, device=DEV),
                    loss=torch.empty(1, device=DEV),
                    ws=torch.empty(gs.mlp_bwd_workspace(S, case["per"]), dtype=torch.uint8, device=DEV))
    if kind == "update":
        p, grads, m, v2, img, target = _update_inputs(case, seed)
        return dict(kind=kind, n=case["n"], degree=case["degree"], p=p, grads=grads, m=m, v=v2, img=img,
                    target=target, partials=torch.empty(gs.L1_PARTIALS, device=DEV), step=10)
    if kind == "density":
        g = _rand(seed)
        n = case["n"]
        p = _scene(g, n, 3, "skewed")
        noise = torch.cat([_normal(g, 3, n), _uniform(g, 3, n, lo=-1.0, hi=1.0)])
        cap = 2 * n
        out = {k: torch.zeros(v.shape[:-1] + (cap,), device=DEV) for k, v in p.items()}
        return dict(kind=kind, n=n, radius=case["radius"], p=p, noise=noise, out=out, cap=cap,
                    g=gs.gaussians_struct(*(p[k] for k in PARAMS), 3),
                    ws=torch.empty(gs.density_control_workspace(n), dtype=torch.uint8, device=DEV))
    raise ValueError(kind)


def run(st):
    kind = st["kind"]
    if kind == "step":
        p, rast = st["p"], st["rast"]
        geometry = (p["means"], p["log_scales"], p["quats"], p["logits"])
        if "dec" in st:
            image = rasterize_learned(*geometry, st["dec"], rast)
        else:
            image = rasterize(*geometry, p["sh"], rast)
        return dict(image=image.detach(), grads=torch.autograd.grad(image, st["leaves"], st["G"]))
    if kind == "render":
        with torch.no_grad():
            return dict(image=rasterize(*(st["p"][k] for k in PARAMS), st["rast"]))
    if kind == "distil":
        gs.mlp_bwd(st["S"], st["per"], st["z"], st["dirs"], st["packed"], st["dlat"], st["dw"], st["ws"],
                   target=st["target"], scale=1.0 / st["S"], loss=st["loss"])
        return dict(latents=st["dlat"], weights=st["dw"], loss=st["loss"])
    if kind == "update":
        loss, dimg = l1_loss(st["img"], st["target"], st["partials"])
        gs.adam_gaussians(st["n"], st["degree"], st["p"], st["grads"], st["m"], st["v"], LRS, st["step"])
        return dict(loss=loss, dimage=dimg, params=st["p"], m=st["m"], v=st["v"])
    if kind == "density":
        rep = gs.density_control(st["g"], dict(radius=st["radius"]), st["noise"], st["out"], st["cap"], st["ws"])
        return dict(report=rep, out=st["out"])
    raise ValueError(kind)


# ----------------------------------------------------------------- least work


def work(case):
    kind = case["kind"]
    if kind == "distil":
        S = case["n"] * case["per"]
        return dict(bytes=S * 24 + case["n"] * (32 + 64) + 6467 * 6, flops=S * 38_000)
    n = case["n"]
    if kind == "density":
        return dict(bytes=n * 236 * 2 + n * 24, flops=n * 200 * 8)
    per = 44 + 12 * (case["degree"] + 1) ** 2
    px = case["width"] * case["height"]
    if kind == "update":
        return dict(bytes=n * per * 7 + px * 36, flops=n * per // 4 * 12)
    colour = 32 if case.get("learned") else per - 44
    fwd = n * (44 + colour) + px * 12
    flops = px * (WALKED * 14 + BLENDED * 10) + n * 500 + (n * 12_700 if case.get("learned") else 0)
    if kind == "render":
        return dict(bytes=fwd, flops=flops)
    colour_out = 64 if case.get("learned") else per - 44
    bwd_flops = px * (WALKED * 14 + BLENDED * 52) + n * 900 + (n * 25_400 if case.get("learned") else 0)
    return dict(bytes=fwd + px * 12 + n * (44 + colour_out), flops=flops + bwd_flops)


# --------------------------------------------------- the same in 64 bits


def _sh_basis(d, degree):
    """Real spherical harmonics with the Condon-Shortley phase at the unit directions d[..., 3]."""
    x, y, z = d.unbind(-1)
    pi = math.pi
    Y = [torch.full_like(x, 0.5 / math.sqrt(pi))]
    if degree > 0:
        a = math.sqrt(3 / (4 * pi))
        Y += [-a * y, a * z, -a * x]
    if degree > 1:
        a, c, e = math.sqrt(15 / pi) / 2, math.sqrt(5 / pi) / 4, math.sqrt(15 / pi) / 4
        Y += [a * x * y, -a * y * z, c * (2 * z * z - x * x - y * y), -a * x * z, e * (x * x - y * y)]
    if degree > 2:
        a, b = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2
        c, e, f = math.sqrt(21 / (2 * pi)) / 4, math.sqrt(7 / pi) / 4, math.sqrt(105 / pi) / 4
        q = 4 * z * z - x * x - y * y
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * q, e * z * (2 * z * z - 3 * x * x - 3 * y * y),
              -c * x * q, f * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, -1)


def _mlp(x, w):
    """The decoder 32 -> 64 -> 64 -> 3 on rows of x, weights in the library's order."""
    sizes = (64 * 32, 64, 64 * 64, 64, 3 * 64, 3)
    W1, b1, W2, b2, W3, b3 = torch.split(w, sizes)
    h = torch.relu(x @ W1.view(64, 32).T + b1)
    h = torch.relu(h @ W2.view(64, 64).T + b2)
    return torch.sigmoid(h @ W3.view(3, 64).T + b3)


def _project64(p, cam, degree, latents=None, weights=None):
    """Records (u, v, conic, opacity, colour) [n][9] with their graph, and depth, radius and liveness."""
    f64 = dict(dtype=torch.float64, device=DEV)
    R, t = torch.tensor(cam.R_cw, **f64), torch.tensor(cam.t_cw, **f64)
    m, q = p["means"], p["quats"] / p["quats"].norm(dim=0, keepdim=True)
    w, x, y, z = q
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).view(-1, 3, 3)
    M = rot * p["log_scales"].exp().T[:, None, :]
    tc = R @ m + t[:, None]
    tz = tc[2]
    live = (tz > cam.near_z).detach()
    tz = torch.where(live, tz, torch.ones_like(tz))
    lx, ly = 1.3 * cam.tan_half_fov_x, 1.3 * cam.tan_half_fov_y
    sx, sy = (tc[0] / tz).clamp(-lx, lx), (tc[1] / tz).clamp(-ly, ly)
    j0 = cam.fx / tz[:, None] * (R[0] - sx[:, None] * R[2])
    j1 = cam.fy / tz[:, None] * (R[1] - sy[:, None] * R[2])
    a0, a1 = (j0[:, None, :] @ M)[:, 0], (j1[:, None, :] @ M)[:, 0]
    a, b, c = (a0 * a0).sum(1) + 0.3, (a0 * a1).sum(1), (a1 * a1).sum(1) + 0.3
    det = a * c - b * b
    u, v = cam.fx * tc[0] / tz + cam.cx, cam.fy * tc[1] / tz + cam.cy
    centre = -R.T @ t
    d = (m - centre[:, None]).T
    Y = _sh_basis(d / d.norm(dim=1, keepdim=True), 3 if latents is not None else degree)
    if latents is not None:
        colour = _mlp(torch.cat([latents, Y], 1), weights)
    else:
        colour = (0.5 + torch.einsum("ij,jci->ic", Y, p["sh"])).clamp(min=0.0)
    rec = torch.cat([torch.stack([u, v, c / det, -b / det, a / det, torch.sigmoid(p["logits"])], 1), colour], 1)
    with torch.no_grad():
        lam = 0.5 * (a + c) + (0.25 * (a - c) ** 2 + b * b).clamp(min=0.1).sqrt()
        radius = torch.ceil(3 * lam.sqrt())
        live = live & (det > 0) & (radius <= 2.0 ** 22)
    return rec, tz.detach(), radius, live


def _tile_lists(rec, depth, radius, live, cam):
    """(tile, Gaussian) entries in (tile, depth) order and every tile's start; None where there are too many."""
    tx, ty = (cam.width + 15) // 16, (cam.height + 15) // 16
    u, v = rec[:, 0], rec[:, 1]
    live = live & (u >= -radius) & (u < 16 * tx + radius) & (v >= -radius) & (v < 16 * ty + radius)
    u, v, r = (torch.where(live, t, torch.zeros_like(t)) for t in (u, v, radius))
    x0, x1 = (torch.floor((u.floor() - r) / 16)).clamp(min=0), (torch.floor((u.floor() + r) / 16)).clamp(max=tx - 1)
    y0, y1 = (torch.floor((v.floor() - r) / 16)).clamp(min=0), (torch.floor((v.floor() + r) / 16)).clamp(max=ty - 1)
    w, h = (x1 - x0 + 1).long(), (y1 - y0 + 1).long()
    cnt = torch.where(live & (w > 0) & (h > 0), w * h, torch.zeros_like(w))
    total = int(cnt.sum())
    if total > 30_000_000:
        return None
    order = torch.argsort(depth)
    cnt = cnt[order]
    gid = torch.repeat_interleave(order, cnt)
    k = torch.arange(total, device=DEV) - torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
    tile = (y0[gid].long() + k // w[gid]) * tx + x0[gid].long() + k % w[gid]
    tile, by = torch.sort(tile, stable=True)
    start = torch.searchsorted(tile, torch.arange(tx * ty + 1, device=DEV))
    return gid[by], start


def _composite64(rec, gid, start, cam, G):
    """The image, and (with G = dL/dimage) dL/drecords, tile group by tile group."""
    tx, ty = (cam.width + 15) // 16, (cam.height + 15) // 16
    image = torch.zeros((3, ty * 16, tx * 16), dtype=torch.float64, device=DEV)
    bg = torch.tensor(cam.bg, dtype=torch.float64, device=DEV)
    grad = torch.zeros_like(rec) if G is not None else None
    if G is not None:
        Gp = torch.zeros_like(image)
        Gp[:, :cam.height, :cam.width] = G
    length = start[1:] - start[:-1]
    order = torch.argsort(length)
    sizes = length[order].tolist()
    ax = torch.arange(16, device=DEV)
    at = 0
    while at < len(sizes):
        end = at + 1
        while end < len(sizes) and (end + 1 - at) * max(sizes[end], 1) * 256 <= 12_000_000:
            end += 1
        tiles, L = order[at:end], max(sizes[end - 1], 1)
        at = end
        px = ((tiles % tx) * 16)[:, None] + ax[None, :]
        py = ((tiles // tx) * 16)[:, None] + ax[None, :]
        X = (px[:, None, :] + 0.5).expand(-1, 16, -1).reshape(len(tiles), 1, 256).double()
        Yc = (py[:, :, None] + 0.5).expand(-1, -1, 16).reshape(len(tiles), 1, 256).double()
        k = torch.arange(L, device=DEV)[None, :]
        have = k < length[tiles][:, None]
        ids = gid[torch.where(have, start[:-1][tiles][:, None] + k, torch.zeros_like(k)).clamp(max=max(len(gid) - 1, 0))] \
            if len(gid) else torch.zeros((len(tiles), L), dtype=torch.long, device=DEV)
        r = rec[ids].detach().requires_grad_(G is not None)
        with torch.set_grad_enabled(G is not None):
            f = [r[..., i, None] for i in range(9)]
            dx, dy = f[0] - X, f[1] - Yc
            power = -0.5 * (f[2] * dx * dx + f[4] * dy * dy) - f[3] * dx * dy
            alpha = (f[5] * power.exp()).clamp(max=0.99)
            keep = (have[..., None] & (power <= 0) & (alpha >= 1.0 / 255.0)).detach()
            alpha = torch.where(keep, alpha, torch.zeros_like(alpha))
            logt = torch.log1p(-alpha)
            incl = logt.cumsum(1)
            blend = (incl.detach() >= math.log(1e-4)).double()  # the walk ends before the entry that goes below
            weight = alpha * (incl - logt).exp() * blend
            T = (logt * blend).sum(1).exp()
            out = torch.stack([(weight * f[6 + c]).sum(1) + T * bg[c] for c in range(3)])
        rows = py[:, :, None].expand(-1, -1, 16).reshape(len(tiles), 256)
        cols = px[:, None, :].expand(-1, 16, -1).reshape(len(tiles), 256)
        image[:, rows, cols] = out.detach()
        if G is not None:
            (g,) = torch.autograd.grad(out, r, Gp[:, rows, cols])
            grad.index_add_(0, ids[have], g[have])
    return image[:, :cam.height, :cam.width], grad


def _exact_frame(case, seed):
    p, G, dec = _frame_inputs(case, seed)
    cam = _camera(case, seed)
    step = case["kind"] == "step"
    p = {k: v.double().requires_grad_(step) for k, v in p.items()}
    z = w = None
    if dec is not None:
        (z, _), (w, _) = dec
        z, w = z.double().requires_grad_(True), w.double().requires_grad_(True)
    rec, depth, radius, live = _project64(p, cam, case["degree"], z, w)
    lists = _tile_lists(rec.detach(), depth, radius, live, cam)
    if lists is None:
        return None
    image, grad = _composite64(rec.detach(), *lists, cam, G.double() if step else None)
    if not step:
        return dict(image=image)
    leaves = [p[k] for k in PARAMS[:4]] + ([z, w] if z is not None else [p["sh"]])
    # a record that is not live has no finite graph to speak of and no gradient
    return dict(image=image, grads=torch.autograd.grad(rec, leaves, grad))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "render"):
        # the colour-hash mode has no value of its own in 64 bits: its groups are decided in 32
        return None if case.get("hashed") else _exact_frame(case, seed)
    if kind == "distil":
        (z, _), (w, _), dirs, target = _distil_inputs(case, seed)
        z, w = z.double().requires_grad_(True), w.double().requires_grad_(True)
        x = torch.cat([z.repeat_interleave(case["per"], 0), _sh_basis(dirs.double(), 3)], 1)
        loss = (_mlp(x, w) - target.double()).square().sum() / len(x)
        return dict(latents=(g := torch.autograd.grad(loss, (z, w)))[0], weights=g[1], loss=loss.detach().reshape(1))
    if kind == "update":
        p, grads, m, v, img, target = _update_inputs(case, seed)
        p, grads, m, v = ({k: t.double() for k, t in d.items()} for d in (p, grads, m, v))
        lr = {k: LRS.get(k) for k in p}
        b1, b2, eps, step = 0.9, 0.999, 1e-15, 10
        for k in p:
            m[k] = b1 * m[k] + (1 - b1) * grads[k]
            v[k] = b2 * v[k] + (1 - b2) * grads[k] ** 2
            d = (m[k] / (1 - b1 ** step)) / ((v[k] / (1 - b2 ** step)).sqrt() + eps)
            if k == "sh":
                d[0] *= LRS["sh_dc"]
                d[1:] *= LRS["sh_rest"]
            else:
                d *= lr[k]
            p[k] = p[k] - d
        diff = img.double() - target.double()
        return dict(loss=diff.abs().mean().reshape(1), dimage=diff.sign() / diff.numel(), params=p, m=m, v=v)
    return None  # density control's decisions are taken in 32 bits
