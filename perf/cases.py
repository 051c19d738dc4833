"""Performance cases of the library: the work its users have it do.

The sizes are those of the seeded workloads of ``paper_2602_12314_amd/scenes.py``
and of ``bench.py`` (a tiny 80x60 image, the 640x480 room, the 1200x680 hall,
eight views of a local map, the 1200x680 keyframe of a 2M-Gaussian map and
their dictionaries), with ragged neighbours of them.  Every case goes through
``paper_2602_12314_amd.ops``:

  render   Renderer.forward + Renderer.backward for a given dL/dQ (Eq. 4)
  rgbd     the same pass with colour and depth, its L1 and SSIM losses and the
           backward of all of them (Eq. 7-9)
  step     one optimisation step by autograd: RenderQueries, DecodeLoss, and
           the gradients of the Gaussians and of the dictionary (Alg. 1, Stage I)
  loss     Decoder.loss_and_grads on a given query map (Eq. 5-6; Stage II
           without dQ)
  infer    Decoder.forward (Eq. 5, the inference decode)
  adjoint  Decode.apply and its backward for a given dL/dF
  tied     TiedDecoder.loss_and_grads (Eq. 5-6 as printed)
  assign   kmeans_assign: nearest dictionary atom of every embedding
  kmeans   StreamKMeans.step: the dictionary initialisation of a keyframe (Eq. 10)

``exact`` is the same mathematics in float64 with torch alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_12314_amd import _lib, ops

DEV = "cuda"
LAMBDA_TR = 0.1
N_PROTO, NOISE = 32, 0.05   # target map: prototypes plus noise, as the scenes draw it
MICRO = 5                   # micro-centres per dictionary atom
QUERY_SCALE = 0.56          # spread of a rendered query component


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # a small crop or a unit-test scene: latency and launches only
        dict(name="render_tiny", kind="render", N=1000, width=80, height=60, views=1, d=16, density=125.0,
             tile_w=16, tile_h=16),
        # the ordinary keyframe of a room-sized map
        dict(name="render_room", kind="render", N=100_000, width=640, height=480, views=1, d=16, density=390.0,
             tile_w=16, tile_h=16),
        # several keyframes of uneven size over a local map in one call
        dict(name="render_views", kind="render", N=500_000, width=1200, height=680, views=8, d=16, density=556.0,
             tile_w=16, tile_h=16),
        # the largest map, with the tile shape the autotuner takes there
        dict(name="render_multifloor", kind="render", N=2_000_000, width=1200, height=680, views=1, d=32,
             density=156.0, tile_w=8, tile_h=32),
        # mapping with colour and depth in the same pass, and the photometric losses
        dict(name="rgbd_hall", kind="rgbd", N=300_000, width=1200, height=680, views=1, d=32, density=333.0,
             tile_w=16, tile_h=16),
        # the whole optimisation step of the 640x480 keyframe
        dict(name="step_room", kind="step", N=100_000, width=640, height=480, views=1, d=16, density=390.0,
             tile_w=16, tile_h=16, prec="bf16", M=256, D=512, shape="px32"),
        # the decode of the tiny image in full precision: latency
        dict(name="loss_tiny_fp32", kind="loss", n=4800, d=16, M=64, D=512, prec="fp32", want_dQ=True, shape="px32"),
        # the largest decode, in the precision and block shape it is run with
        dict(name="loss_multifloor_fp8", kind="loss", n=816_000, d=32, M=1024, D=1024, prec="fp8", want_dQ=True,
             shape="px64"),
        # serving: dense features of one ragged image from a dictionary that fills no whole tile
        dict(name="infer_hall_bf16", kind="infer", n=307_201, d=32, M=500, D=768, prec="bf16", shape="px32"),
        # a user's own loss on F: decode and its adjoint through autograd, on a ragged crop
        dict(name="adjoint_crop_bf16", kind="adjoint", n=76_799, d=32, M=512, D=768, prec="bf16", shape="px64"),
        # the decode and loss as the paper prints them
        dict(name="tied_hall_bf16", kind="tied", n=816_000, d=32, M=512, D=768, prec="bf16", shape="px64"),
        # the dictionary of a keyframe by streaming K-means
        dict(name="kmeans_keyframe_bf16", kind="kmeans", n=307_200, D=512, K=256, prec="bf16", iters=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render", "render", "rgbd", "step", "loss", "loss", "infer", "adjoint", "tied", "assign", "kmeans"])
    c = dict(kind=kind)
    if kind in ("render", "rgbd", "step"):
        views = rng.choice([1, 1, 2, 3, 5]) if kind == "render" else 1
        w = _log_int(rng, 80, 1200)
        c.update(N=_log_int(rng, 1000, 1_500_000 // views), width=w, height=max(48, int(w * rng.uniform(0.5, 0.8))),
                 views=views, d=rng.choice([16, 32]), density=round(rng.uniform(125.0, 450.0), 1))
        c["tile_w"], c["tile_h"] = rng.choice([(16, 16), (16, 16), (8, 32), (32, 8), (16, 8), (8, 8)])
        if kind == "step":
            c.update(prec=rng.choice(["bf16", "fp32"]), M=_log_int(rng, 32, 1024), D=128 * rng.randint(1, 8),
                     shape=rng.choice(["px32", "px64"]))
        return c
    if kind in ("loss", "infer", "adjoint", "tied"):
        prec = rng.choice(["bf16", "bf16", "fp32"] if kind == "tied" else ["bf16", "fp8", "fp32"])
        c.update(n=_log_int(rng, 1000, 200_000 if prec == "fp32" else 816_000), d=rng.choice([16, 32]),
                 M=_log_int(rng, 32, 1024), D=128 * rng.randint(1, 8), prec=prec, shape=rng.choice(["px32", "px64"]))
        if kind == "loss":
            c["want_dQ"] = rng.random() < 0.7
        return c
    prec = rng.choice(["bf16", "bf16", "fp32"])
    c.update(n=_log_int(rng, 5000, 100_000 if prec == "fp32" else 500_000), D=32 * rng.randint(4, 32),
             K=_log_int(rng, 16, 1000), prec=prec)
    if kind == "kmeans":
        c["K"] = _log_int(rng, 16, 300)
        c["iters"] = rng.choice([3, 5, 10])
    return c


# ------------------------------------------------------------------ inputs

def _cams(case):
    """Camera rows [width, height, fx, fy, cx, cy, viewmat]: one camera at the
    origin looking along z, or ``views`` cameras of uneven size on a circle of
    radius 3 looking at the centre.  Focal length 525 at width 640."""
    W, H, views = case["width"], case["height"], case["views"]
    rows = []
    scale = [0.27, 0.4, 0.53, 0.53, 0.53, 0.8, 1.0, 1.0]
    for k in range(views):
        s = 1.0 if views == 1 else scale[(k * len(scale)) // views]
        w, h = max(16, int(round(W * s))), max(16, int(round(H * s)))
        f = 525.0 * w / 640.0
        vm = np.eye(4)
        if views > 1:
            th = 2.0 * math.pi * k / views
            c = np.array([3.0 * math.cos(th), 0.0, 3.0 * math.sin(th)])
            fwd = -c / np.linalg.norm(c)
            right = np.cross([0.0, 1.0, 0.0], fwd)
            right /= np.linalg.norm(right)
            vm[:3, :3] = np.stack([right, np.cross(fwd, right), fwd])
            vm[:3, 3] = -vm[:3, :3] @ c
        rows.append([w, h, f, f, w / 2, h / 2, *vm.reshape(-1)])
    return np.asarray(rows, np.float32)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(shape, device=DEV, generator=g)


def _rand(g, *shape):
    return torch.rand(shape, device=DEV, generator=g)


def _gaussians(case, g):
    """A map of N Gaussians, 4 m high (8 m beyond a million: several floors) and
    as wide as the density asks, in front of the camera or around the origin."""
    N = case["N"]
    height = min(8.0 if N > 1_000_000 else 4.0, (N / case["density"]) ** (1.0 / 3.0))
    side = math.sqrt(N / (case["density"] * height))
    around = case["views"] > 1 or N > 1_000_000
    u = _rand(g, N, 3)
    lo = torch.tensor([-side / 2, -height / 2, -side / 2 if around else 0.5], device=DEV)
    means = lo + u * torch.tensor([side, height, side], device=DEV)
    log_scales = -3.0 + 0.3 * _randn(g, N, 3)
    quats = torch.nn.functional.normalize(_randn(g, N, 4), dim=1)
    return [means, log_scales, quats, _randn(g, N), _randn(g, N, case["d"])]


def _target(g, n, D):
    """Rows of unit norm: one of 32 prototypes, constant over runs of pixels, plus noise."""
    protos = torch.nn.functional.normalize(_randn(g, N_PROTO, D), dim=1)
    runs = torch.randint(0, N_PROTO, (n // 40 + 1,), device=DEV, generator=g)
    t = protos[runs.repeat_interleave(40)[:n]]
    t += NOISE * _randn(g, n, D)
    return torch.nn.functional.normalize(t, dim=1)


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("render", "rgbd", "step"):
        s["cams"] = _cams(case)
        s["params"] = _gaussians(case, g)
        n = int((s["cams"][:, 0] * s["cams"][:, 1]).sum())
        if kind != "step":
            s["dQ"] = _randn(g, n, case["d"]) / n
    if kind == "rgbd":
        s["colors"] = _rand(g, case["N"], 3)
        s["rgb_obs"] = _rand(g, n, 3)
        depth = 0.5 + 8.0 * _rand(g, n)
        s["depth_obs"] = torch.where(_rand(g, n) < 0.1, torch.zeros_like(depth), depth)  # sensors leave holes
    if kind in ("loss", "infer", "adjoint", "tied", "step"):
        if kind != "step":
            n = case["n"]
            s["Q"] = QUERY_SCALE * _randn(g, n, case["d"])
        M, D, d = case["M"], case["D"], case["d"]
        s["K"], s["V"] = _randn(g, M, d), _randn(g, M, D)
        s["K0"] = s["K"] + 0.01 * _randn(g, M, d)
        if kind == "adjoint":
            s["dF"] = _randn(g, n, D) / n
        elif kind != "infer":
            s["target"] = _target(g, n, D)
        if kind == "tied":
            s["W"] = _randn(g, d, D) / math.sqrt(d)
            s["V0"] = s["V"] + 0.01 * _randn(g, M, D)
    if kind in ("assign", "kmeans"):
        s["F"] = _target(g, case["n"], case["D"])
        if kind == "assign":
            s["C"] = s["F"][torch.randperm(case["n"], device=DEV, generator=g)[:case["K"]]].clone()
        else:
            m = min(case["n"], MICRO * case["K"])
            s["seeds"] = np.random.default_rng(seed).choice(case["n"], size=m, replace=False).astype(np.int32)
            s["D_prev"] = s["F"][torch.randperm(case["n"], device=DEV, generator=g)[:case["K"] // 2]].clone()
            s["W_prev"] = 1.0 + 100.0 * _rand(g, case["K"] // 2)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("render", "rgbd", "step"):
        s["g"] = ops.Gaussians(*s["params"])
        s["renderer"] = ops.Renderer(s["cams"], case["N"], case["d"], tile=(case["tile_w"], case["tile_h"]))
    if kind == "step":
        s["params"] = [t.requires_grad_(True) for t in s["params"]]
        s["dict"] = [s["K"].requires_grad_(True), s["V"].requires_grad_(True)]
    if kind in ("loss", "infer", "adjoint", "tied", "step"):
        s["ctx"] = _lib.Context(options={"decode_shape": case["shape"]})
        n = s["target"].shape[0] if kind == "step" else case["n"]
        cls = ops.TiedDecoder if kind == "tied" else ops.Decoder
        s["dec"] = cls(case["prec"], n, case["d"], case["M"], case["D"], device=DEV, ctx=s["ctx"])
    if kind == "adjoint":
        s["leaves"] = [s[k].requires_grad_(True) for k in ("Q", "K", "V")]
    if kind == "kmeans":
        s["km"] = ops.StreamKMeans(case["prec"], case["K"], case["D"], iters_local=case["iters"],
                                   iters_global=case["iters"], device=DEV)
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "render":
        Q, T = s["renderer"].forward(s["g"])
        grads = s["renderer"].backward(s["g"], s["dQ"])
        return dict(Q=Q, T=T, grads=list(grads.tensors()))
    if kind == "rgbd":
        r, g = s["renderer"], s["g"]
        Q, rgb, depth, T = r.forward_rgbd(g, s["colors"])
        l1, d_rgb, d_depth = ops.rgbd_l1_loss(rgb, s["rgb_obs"], depth, s["depth_obs"])
        ls, d_rgb = ops.ssim_loss(rgb, s["rgb_obs"], s["cams"], d_rgb=d_rgb)
        grads, d_colors = r.backward_rgbd(g, s["colors"], s["dQ"], d_rgb, d_depth)
        return dict(Q=Q, rgb=rgb, depth=depth, T=T, l1=l1, ssim=ls, grads=list(grads.tensors()), d_colors=d_colors)
    if kind == "step":
        Q, T = ops.RenderQueries.apply(s["renderer"], *s["params"])
        loss = ops.DecodeLoss.apply(Q, *s["dict"], s["K0"], s["target"], LAMBDA_TR, s["dec"])
        grads = torch.autograd.grad(loss, s["params"] + s["dict"])
        return dict(Q=Q.detach(), T=T, loss=loss.detach(), grads=list(grads))
    if kind == "loss":
        loss, dQ, dK, dV = s["dec"].loss_and_grads(s["Q"], s["K"], s["V"], s["target"], s["K0"], LAMBDA_TR,
                                                   want_dQ=case["want_dQ"])
        return dict(loss=loss, dQ=dQ, dK=dK, dV=dV)
    if kind == "infer":
        return s["dec"].forward(s["Q"], s["K"], s["V"])
    if kind == "adjoint":
        F = ops.Decode.apply(*s["leaves"], s["dec"])
        dQ, dK, dV = torch.autograd.grad(F, s["leaves"], s["dF"])
        return dict(F=F.detach(), dQ=dQ, dK=dK, dV=dV)
    if kind == "tied":
        loss, dQ, dW, dD = s["dec"].loss_and_grads(s["Q"], s["W"], s["V"], s["target"], s["V0"])
        return dict(loss=loss, dQ=dQ, dW=dW, dD=dD)
    if kind == "assign":
        a, d2 = ops.kmeans_assign(case["prec"], s["F"], s["C"])
        return dict(assign=a, d2=d2)
    km = s["km"]  # the keyframe is merged into the dictionary of the keyframes before
    km.D, km.W = s["D_prev"], s["W_prev"]
    D, W = km.step(s["F"], seeds=s["seeds"])
    return dict(D=D, W=W)


# ------------------------------------------------------------------ work

def work(case):
    """Bytes: every input read and every output written once (float32).  Flops:
    the method's products; for the renders only the projection of every record
    and its adjoint, since how many (Gaussian, pixel) pairs blend depends on
    the scene."""
    kind = case["kind"]
    byts = flops = 0.0
    n = case.get("n", 0)
    if kind in ("render", "rgbd", "step"):
        cams = _cams(case)
        n = float((cams[:, 0] * cams[:, 1]).sum())
        N, d = case["N"], case["d"]
        byts += 4.0 * (2 * N * (11 + d) + n * (2 * d + 1))  # parameters and gradients; Q, T, dQ
        flops += 900.0 * N * case["views"]
        if kind == "rgbd":
            byts += 4.0 * (2 * 3 * N + n * (4 + 4 + 4))
            flops += n * 3 * 2.0 * 8 * 22
    if kind in ("loss", "infer", "adjoint", "tied", "step"):
        d, M, D = case["d"], case["M"], case["D"]
        byts += 4.0 * (n * D + (0 if kind == "step" else n * d) + M * (d + D))
        if kind == "infer":
            flops += 2.0 * n * M * (d + D)
        else:
            byts += 4.0 * M * (d + D)
            if kind != "step" and case.get("want_dQ", True):
                byts += 4.0 * n * d
            flops += 6.0 * n * M * (d + D)
        if kind == "adjoint":
            byts += 4.0 * n * D
        if kind == "tied":
            byts += 4.0 * (M * D + 2 * d * D)
            flops += 6.0 * M * d * D + 6.0 * n * d * d
    if kind == "assign":
        byts = 4.0 * (n * case["D"] + case["K"] * case["D"] + 2 * n)
        flops = 2.0 * n * case["K"] * case["D"]
    if kind == "kmeans":
        K, D, it = case["K"], case["D"], case["iters"]
        m = min(n, MICRO * K)
        byts = 4.0 * (n * D + (K + K // 2) * (D + 1))
        flops = 2.0 * it * D * (n * m + (K // 2 + m) * K)
    return dict(bytes=byts, flops=flops)


# ------------------------------------------------------------------ float64

def _exact_project(cam, means, log_scales, quats, logits):
    """Visible records of one camera: indices, footprints and the float64
    quantities (u, v, conic A B C, opacity, z), differentiable in the inputs."""
    w, h, fx, fy, cx, cy = (float(v) for v in cam[:6])
    vm = torch.as_tensor(cam[6:], dtype=torch.float64, device=DEV).reshape(4, 4)
    Wr, t = vm[:3, :3], vm[:3, 3]
    near = torch.nonzero((means.detach() @ Wr.T + t)[:, 2] > 0.2).flatten()
    p = means[near] @ Wr.T + t
    x, y, z = p.unbind(1)
    q = quats[near]
    q = q / q.norm(dim=1, keepdim=True)
    a, b, c, e = q.unbind(1)
    R = torch.stack([1 - 2 * (c * c + e * e), 2 * (b * c - a * e), 2 * (b * e + a * c),
                     2 * (b * c + a * e), 1 - 2 * (b * b + e * e), 2 * (c * e - a * b),
                     2 * (b * e - a * c), 2 * (c * e + a * b), 1 - 2 * (b * b + c * c)], 1).reshape(-1, 3, 3)
    Mx = Wr @ (R * torch.exp(log_scales[near])[:, None, :])
    lx, ly = 1.3 * w / (2 * fx), 1.3 * h / (2 * fy)
    tx, ty = (x / z).clamp(-lx, lx), (y / z).clamp(-ly, ly)
    r0 = (fx / z)[:, None] * (Mx[:, 0] - tx[:, None] * Mx[:, 2])
    r1 = (fy / z)[:, None] * (Mx[:, 1] - ty[:, None] * Mx[:, 2])
    ca, cb, cc = (r0 * r0).sum(1) + 0.3, (r0 * r1).sum(1), (r1 * r1).sum(1) + 0.3
    det = ca * cc - cb * cb
    u, v = fx * x / z + cx, fy * y / z + cy
    with torch.no_grad():
        mid = 0.5 * (ca + cc)
        rad = torch.ceil(3.0 * torch.sqrt(mid + torch.sqrt((mid * mid - det).clamp(min=0.1))))
        x0, x1 = torch.ceil(u - rad).clamp(min=0), torch.floor(u + rad).clamp(max=w - 1)
        y0, y1 = torch.ceil(v - rad).clamp(min=0), torch.floor(v + rad).clamp(max=h - 1)
        vis = torch.nonzero((x0 <= x1) & (y0 <= y1)).flatten()
    rec = torch.stack([u, v, cc / det, -cb / det, ca / det, torch.sigmoid(logits[near]), z], 1)[vis]
    box = torch.stack([x0, x1, y0, y1], 1)[vis].to(torch.int64)
    return near[vis], box, rec


def _exact_lists(case_w, case_h, box, z, T=16):
    """Per 16x16 tile, the records whose footprint touches it, nearest first:
    (records sorted by tile and depth, start of each tile, tiles per row)."""
    tx = (case_w + T - 1) // T
    ty = (case_h + T - 1) // T
    order = torch.argsort(z.float(), stable=True)
    bx = box[order] // T
    nx, ny = bx[:, 1] - bx[:, 0] + 1, bx[:, 3] - bx[:, 2] + 1
    cnt = nx * ny
    who = torch.repeat_interleave(torch.arange(len(order), device=DEV), cnt)
    k = torch.arange(len(who), device=DEV) - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
    tile = (bx[who, 2] + k // nx[who]) * tx + bx[who, 0] + k % nx[who]
    by_tile = torch.argsort(tile, stable=True)
    start = torch.searchsorted(tile[by_tile], torch.arange(tx * ty + 1, device=DEV))
    return order[who[by_tile]], start, tx


def _exact_blend(cam, box, rec, val, upstream):
    """Blends val [R, C] into the image of one camera: (image [P, C], T [P]).
    With upstream [P, C], adds d(sum upstream * image) to rec.grad and val.grad
    instead."""
    w, h = int(cam[0]), int(cam[1])
    T, C = 16, val.shape[1]
    lst, start, tx = _exact_lists(w, h, box, rec.detach()[:, 6])
    length = (start[1:] - start[:-1]).cpu().numpy()
    image = torch.zeros(w * h, C, dtype=torch.float64, device=DEV)
    trans = torch.ones(w * h, dtype=torch.float64, device=DEV)
    tiles = np.argsort(-length, kind="stable")
    tiles = tiles[length[tiles] > 0]
    at, lane = 0, torch.arange(T * T, device=DEV)
    while at < len(tiles):
        L = int(length[tiles[at]])
        some = torch.as_tensor(tiles[at:at + max(1, 40_000_000 // (256 * L))], device=DEV)
        at += len(some)
        k = torch.arange(L, device=DEV)
        idx = start[some][:, None] + k
        have = k < (start[some + 1] - start[some])[:, None]
        idx = lst[idx.clamp(max=len(lst) - 1)]
        px = (some % tx)[:, None] * T + lane % T
        py = torch.div(some, tx, rounding_mode="floor")[:, None] * T + lane // T
        inside = (px < w) & (py < h)
        b = box[idx][:, None]
        ok = have[:, None] & (px[..., None] >= b[..., 0]) & (px[..., None] <= b[..., 1])
        ok &= (py[..., None] >= b[..., 2]) & (py[..., None] <= b[..., 3])
        with torch.set_grad_enabled(upstream is not None):
            r = rec[idx][:, None]
            dx, dy = r[..., 0] - px[..., None], r[..., 1] - py[..., None]
            power = -0.5 * (r[..., 2] * dx * dx + r[..., 4] * dy * dy) - r[..., 3] * dx * dy
            alpha = (r[..., 5] * torch.exp(power)).clamp(max=0.99)
            alpha = torch.where(ok & (alpha >= 1.0 / 255.0), alpha, torch.zeros_like(alpha))
            cum = torch.cumprod(1.0 - alpha, -1)
            alive = cum >= 1e-4
            before = torch.cat([torch.ones_like(cum[..., :1]), cum[..., :-1]], -1)
            wgt = torch.where(alive, alpha * before, torch.zeros_like(alpha))
            out = torch.matmul(wgt, val[idx])
        pix = (py * w + px)[inside]
        if upstream is None:
            image[pix] = out[inside]
            left = torch.where(alive, cum, torch.full_like(cum, 2.0)).amin(-1)
            trans[pix] = torch.where(left > 1.5, torch.ones_like(left), left)[inside]
        else:
            torch.autograd.backward(out[inside], upstream[pix])
    return image, trans


class _ExactRender:
    """Float64 render of all cameras; val = [queries | extra channels]."""

    def __init__(self, cams, params, colors=None):
        self.cams = cams
        self.leaves = [t.detach().double().requires_grad_(True) for t in params + ([] if colors is None else [colors])]
        means, log_scales, quats, logits, queries = self.leaves[:5]
        self.parts = []
        for cam in cams:
            who, box, rec = _exact_project(cam, means, log_scales, quats, logits)
            val = queries[who]
            if colors is not None:
                val = torch.cat([val, self.leaves[5][who], rec[:, 6:7]], 1)
            self.parts.append((cam, box, rec, val, rec.detach().requires_grad_(True),
                               val.detach().requires_grad_(True)))

    def forward(self):
        got = [_exact_blend(cam, box, r, v, None) for cam, box, _, _, r, v in self.parts]
        return torch.cat([a for a, _ in got]), torch.cat([t for _, t in got])

    def backward(self, up):
        off, outs, grads = 0, [], []
        for cam, box, rec, val, r, v in self.parts:
            n = int(cam[0]) * int(cam[1])
            _exact_blend(cam, box, r, v, up[off:off + n])
            off += n
            if r.grad is not None:
                outs += [rec, val]
                grads += [r.grad, v.grad]
        got = torch.autograd.grad(outs, self.leaves, grads, allow_unused=True) if outs else [None] * len(self.leaves)
        return [torch.zeros_like(t) if x is None else x for t, x in zip(self.leaves, got)]


def _exact_ssim(x, y, cams, lam):
    """lam (1 - SSIM): 11 x 11 Gaussian window, zero padding, per channel and view."""
    k = torch.arange(11, dtype=torch.float64, device=DEV) - 5
    win = torch.exp(-k * k / (2 * 1.5 ** 2))
    win = win / win.sum()

    def blur(im):
        for dim in (0, 1):
            pad = torch.zeros_like(im.narrow(dim, 0, 1)).expand(*[5 if i == dim else n for i, n in enumerate(im.shape)])
            big = torch.cat([pad, im, pad], dim)
            im = sum(win[i] * big.narrow(dim, i, im.shape[dim]) for i in range(11))
        return im

    off, total = 0, 0.0
    for cam in cams:
        w, h = int(cam[0]), int(cam[1])
        a, b = (t[off:off + w * h].reshape(h, w, 3) for t in (x, y))
        off += w * h
        ma, mb = blur(a), blur(b)
        va, vb, vab = blur(a * a) - ma * ma, blur(b * b) - mb * mb, blur(a * b) - ma * mb
        c1, c2 = 0.01 ** 2, 0.03 ** 2
        total = total + (((2 * ma * mb + c1) * (2 * vab + c2)) / ((ma * ma + mb * mb + c1) * (va + vb + c2))).sum()
    return lam * (1.0 - total / (3.0 * off))


def _exact_decode(Q, K, V, scale, row_grad, rows=32768, want_F=False):
    """Attention in float64 a slice of the rows at a time; row_grad(F, rows)
    gives each slice's loss terms and dL/dF.  (loss, F, dQ, dK, dV)"""
    dK, dV = torch.zeros_like(K), torch.zeros_like(V)
    loss, dQ, Fs = 0.0, [], []
    for a in range(0, Q.shape[0], rows):
        s = slice(a, a + rows)
        P = torch.softmax((Q[s] @ K.T) * scale, 1)
        F = P @ V
        if want_F:
            Fs.append(F)
        if row_grad is None:
            continue
        part, G = row_grad(F, s)
        loss = loss + part
        dP = G @ V.T
        dS = P * (dP - (P * dP).sum(1, keepdim=True)) * scale
        dQ.append(dS @ K)
        dK += dS.T @ Q[s]
        dV += P.T @ G
    return loss, torch.cat(Fs) if Fs else None, torch.cat(dQ) if dQ else None, dK, dV


def _cosine_grad(target, n, lam_cos=1.0, lam_2=0.0):
    def of(F, s):
        T = target[s].double()
        nf, nt = F.norm(dim=1, keepdim=True), T.norm(dim=1, keepdim=True)
        cos = (F * T).sum(1, keepdim=True) / (nf * nt)
        G = -lam_cos / n * (T / (nf * nt) - cos * F / (nf * nf)) + 2.0 * lam_2 / n * (F - T)
        return (lam_cos * (1 - cos).sum() + lam_2 * ((F - T) ** 2).sum()) / n, G
    return of


def exact(case, seed):
    kind = case["kind"]
    s = _inputs(case, seed)
    if kind in ("render", "rgbd", "step"):
        d = case["d"]
        r = _ExactRender(s["cams"], s["params"], s.get("colors"))
        image, T = r.forward()
        Q = image[:, :d].contiguous()
    if kind == "render":
        return dict(Q=Q, T=T, grads=r.backward(s["dQ"].double()))
    if kind == "rgbd":
        rgb, depth = image[:, d:d + 3].contiguous(), image[:, d + 3].contiguous()
        obs, dobs = s["rgb_obs"].double(), s["depth_obs"].double()
        with torch.enable_grad():
            x, z = rgb.clone().requires_grad_(True), depth.clone().requires_grad_(True)
            seen = dobs > 0
            l1 = 0.2 * (x - obs).abs().mean() + 0.1 * (z - dobs)[seen].abs().mean()
            ls = _exact_ssim(x, obs, s["cams"], 0.8)
            d_rgb, d_depth = torch.autograd.grad(l1 + ls, (x, z))
        grads = r.backward(torch.cat([s["dQ"].double(), d_rgb, d_depth[:, None]], 1))
        return dict(Q=Q, rgb=rgb, depth=depth, T=T, l1=l1.detach().reshape(1), ssim=ls.detach().reshape(1),
                    grads=grads[:5], d_colors=grads[5])
    if kind in ("loss", "infer", "adjoint", "step"):
        K, V, K0 = s["K"].double(), s["V"].double(), s["K0"].double()
        if kind != "step":
            Q = s["Q"].double()
        scale = 1.0 / math.sqrt(case["d"])
        if kind == "infer":
            return _exact_decode(Q, K, V, scale, None, want_F=True)[1]
        if kind == "adjoint":
            dF = s["dF"]
            _, F, dQ, dK, dV = _exact_decode(Q, K, V, scale, lambda F, q: (0.0, dF[q].double()), want_F=True)
            return dict(F=F, dQ=dQ, dK=dK, dV=dV)
        n = Q.shape[0]
        loss, _, dQ, dK, dV = _exact_decode(Q, K, V, scale, _cosine_grad(s["target"], n))
        loss = loss + LAMBDA_TR * ((K - K0) ** 2).sum()
        dK = dK + 2 * LAMBDA_TR * (K - K0)
        if kind == "step":
            return dict(Q=Q, T=T, loss=loss, grads=r.backward(dQ) + [dK, dV])
        return dict(loss=loss.reshape(1), dQ=dQ if case["want_dQ"] else None, dK=dK, dV=dV)
    if kind == "tied":
        p = dict(tau=0.1, lambda_cos=0.5, lambda_2=0.5, lambda_D=0.2, delta=0.1)
        Q, W, V, V0 = (s[k].double() for k in ("Q", "W", "V", "V0"))
        W.requires_grad_(True)
        V.requires_grad_(True)
        Q.requires_grad_(True)
        # logits = (Q W / |Q W|) (V / |V|)^T / tau = Qs Kt^T with Kt = normalise(V) W^T
        norm = torch.sqrt(((Q @ (W @ W.T)) * Q).sum(1, keepdim=True))
        Qs = Q / (p["tau"] * norm)
        Kt = torch.nn.functional.normalize(V, dim=1) @ W.T
        loss, _, dQs, dKt, dV = _exact_decode(Qs.detach(), Kt.detach(), V.detach(), 1.0,
                                              _cosine_grad(s["target"], Q.shape[0], p["lambda_cos"], p["lambda_2"]))
        hinge = p["lambda_D"] * torch.relu((V0 - V).norm(dim=1) - p["delta"]).sum()
        dQ, dW, dD = torch.autograd.grad((Qs * dQs).sum() + (Kt * dKt).sum() + (V * dV).sum() + hinge, (Q, W, V))
        return dict(loss=(loss + hinge).detach().reshape(1), dQ=dQ, dW=dW, dD=dD)
    if kind == "assign":
        F, C = s["F"], s["C"].double()
        best = []
        for a in range(0, F.shape[0], 32768):
            x = F[a:a + 32768].double()
            best.append(((x * x).sum(1, keepdim=True) - 2.0 * x @ C.T + (C * C).sum(1)).amin(1).clamp(min=0.0))
        return dict(assign=None, d2=torch.cat(best))
    # K-means: which centre a point between two of them goes to is decided by
    # the rounding of the distances, and every later iteration follows from it
    return None
