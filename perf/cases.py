"""Workloads of the Universal Beta Splatting renderer, as its users call it.

A case is one call (or one training iteration up to the optimiser) through
the public entry points of ``paper_2510_03312_amd``:

  view      ``Renderer.forward``: an image served or evaluated, no gradient
  frame     ``Renderer.forward`` and ``Renderer.backward`` with the fused L1 loss
  render    ``render()`` under autograd, gradients given for the image and the
            final transmittance (a program with its own torch loss)
  train     ``Renderer.forward``, ``ssim_loss``, ``Renderer.backward``: a training
            iteration with the L1 + D-SSIM loss up to the optimiser
  replay    ``GraphFrame.replay``: the same frame as ``frame`` from a HIP graph
  ssim      ``ssim_loss`` by itself
  adam      ``adam_step`` by itself (it updates its tensors in place)
  relocate  ``relocate`` by itself, on opacities as an optimiser left them

Scenes follow the distributions of the repository's synthetic workloads:
3-D centres uniform in a cube, N-D centres normal around the origin with
angular, temporal and further query dimensions; cameras on a circle of
radius 4 looking at the origin, 60 degrees of horizontal field of view.
"""
import dataclasses
import math

import numpy as np
import torch

import paper_2510_03312_amd as ubs
from paper_2510_03312_amd.renderer import GraphFrame

QUAT, SKEW = 0, 1
NEAR, DILATION, ALPHA_MIN, ALPHA_MAX, T_STOP = 0.2, 0.3, 1.0 / 255.0, 0.99, 1e-4
LAMBDA_SSIM, O_MIN, ADAM_STEP = 0.2, 0.005, 500
FRAMES = ("view", "frame", "render", "train", "replay")


def listed():
    full = "1920x1080"
    return [
        # the smallest call: a static object of a few thousand primitives in a thumbnail,
        # a program with its own torch loss; launches and host work count
        _frame("small_3d_autograd", "render", 3, "2000", "128x128"),
        # serving a preview from a small dynamic scene, with the float32 option
        _frame("preview_7d_fp32", "view", 7, "100000", "640x480", fp32=True),
        # evaluating a held-out view of a static view-dependent capture
        _frame("view_6d", "view", 6, "500000", "1264x832"),
        # an ordinary training iteration with D-SSIM: odd sizes, the skew rotation
        _frame("train_7d_odd", "train", 7, "250001", "1237x821", rot=SKEW),
        # fwd + bwd at 1080p, view-dependent
        _frame("frame_6d_1080p", "frame", 6, "1000000", full),
        # fwd + bwd at 1080p, dynamic, replayed from a graph (the headline workload)
        _frame("replay_7d_1080p", "replay", 7, "1000000", full),
        # beyond 7-D: three query values given by the view
        _frame("frame_10d_1080p", "frame", 10, "1000000", full),
        # one batch of eight views of one scene
        _frame("views8_7d", "frame", 7, "2000000", "1352x1014", views=8),
        # the largest: several scenes, many views of uneven resolution in one batch
        _frame("scenes4_views32", "frame", 7, "100000,500000,1500000,3000000",
               "640x480,1280x720,1920x1080", views=32),
        # the image loss by itself
        {"name": "ssim_1080p", "kind": "ssim", "res": full, "views": 1},
        # the optimiser step of a full scene
        {"name": "adam_7d_1m", "kind": "adam", "dim": 7, "rot": QUAT, "n": 1000000, "noise": True},
        # densification: 30 % of a full scene dead
        {"name": "relocate_7d_1m", "kind": "relocate", "dim": 7, "rot": QUAT, "n": 1000000,
         "dead": 0.3},
    ]


def _frame(name, kind, dim, sizes, res, *, rot=QUAT, views=1, fp32=False):
    return {"name": name, "kind": kind, "dim": dim, "rot": rot, "sizes": sizes, "res": res,
            "views": views, "fp32": fp32}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _res(rng, pixels):
    aspect = math.exp(rng.uniform(math.log(0.75), math.log(1.9)))
    w = max(64, int(math.sqrt(pixels * aspect)))
    return "%dx%d" % (w, max(48, int(pixels / w)))


def draw(rng):
    kind = rng.choice(FRAMES + FRAMES + ("ssim", "adam", "relocate"))
    if kind == "ssim":
        views = rng.choice((1, 1, 2, 5))
        return {"kind": kind, "views": views,
                "res": ",".join(_res(rng, _log_int(rng, 10000, 2100000)) for _ in range(min(views, 3)))}
    dim = rng.choice((3, 6, 6, 7, 7, 8, 9, 10))
    rot = rng.choice((QUAT, QUAT, SKEW))
    if kind == "adam":
        return {"kind": kind, "dim": dim, "rot": rot, "n": _log_int(rng, 2000, 2000000),
                "noise": rng.random() < 0.7}
    if kind == "relocate":
        return {"kind": kind, "dim": dim, "rot": rot, "n": _log_int(rng, 2000, 2000000),
                "dead": round(rng.uniform(0.01, 0.5), 3)}
    # a static 3-D scene keeps every primitive in view: smaller ones
    n = _log_int(rng, 2000, 300000 if dim == 3 else 2000000)
    views = rng.choice((1, 1, 1, 2, 3, 6))
    sizes = [n] if views == 1 or rng.random() < 0.6 else [n, _log_int(rng, 2000, n + 1)]
    pixels = min(2100000, max(10000, n * math.exp(rng.uniform(math.log(0.7), math.log(8.0)))))
    res = [_res(rng, pixels)] + ([_res(rng, pixels / 2)] if views > 1 and rng.random() < 0.5 else [])
    return {"kind": kind, "dim": dim, "rot": rot, "sizes": ",".join(map(str, sizes)),
            "res": ",".join(res), "views": views, "fp32": rng.random() < 0.15}


# ------------------------------------------------------------------- inputs
@dataclasses.dataclass
class View:
    scene: int
    width: int
    height: int
    R: np.ndarray
    t: np.ndarray
    fx: float
    fy: float
    cx: float
    cy: float
    time: float
    query: tuple


def _rows(dim, rot):
    """First row of every parameter block, and their number."""
    c, k, at = dim - 3, 0, {}
    for name, m in (("mu", 3), ("muq", c), ("rot", 4 if rot == QUAT else 3), ("logs", 3),
                    ("lqx", 3 * c), ("lq", c * (c + 1) // 2), ("bx", 1), ("bq", c), ("o", 1),
                    ("rgb", 3)):
        at[name] = k
        k += m
    return at, k


def _gen(seed, *more):
    g = torch.Generator(device="cuda")
    s = int(seed) * 7919 + 17
    for m in more:
        s = s * 1009 + int(m)
    g.manual_seed(s % (1 << 62))
    return g


def _scene(dim, rot, n, g):
    c = dim - 3

    def U(m, lo=0.0, hi=1.0):
        return torch.rand((m, n), generator=g, device="cuda") * (hi - lo) + lo

    def N(m, mean=0.0, std=1.0):
        return torch.randn((m, n), generator=g, device="cuda") * std + mean

    def unit(x):
        return x / x.norm(dim=0, keepdim=True)

    rows = [U(3, -1.0, 1.0) if c == 0 else N(3, 0.0, 1.5)]
    if c >= 4:
        rows.append(U(1))
    if c:
        rows.append(unit(N(3)))
    if c > 4:
        rows.append(U(c - 4))
    rows.append(unit(N(4)) if rot == QUAT else N(3, 0.0, 0.3))
    rows.append(N(3, -3.0, 0.3))
    if c:
        rows.append(N(3 * c, 0.0, 0.3))
        for i in range(c):
            if i:
                rows.append(N(i, 0.0, 0.1))
            rows.append((U(1, 0.02, 0.5) if c >= 4 and i == 0 else U(1, 0.2, 2.0)).log())
    rows += [U(1 + c, -1.0, 1.0), torch.sigmoid(N(1)), U(3)]
    return torch.cat(rows).contiguous()


def _views(case, seed):
    res = [tuple(int(x) for x in r.split("x")) for r in case["res"].split(",")]
    n_scenes = len(case["sizes"].split(",")) if "sizes" in case else 1
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 5])
    nv, out = int(case["views"]), []
    turn, time0 = rng.uniform(0.0, 2.0 * math.pi), rng.uniform(0.3, 0.7)
    for k in range(nv):
        w, h = res[k % len(res)]
        th = turn + 2.0 * math.pi * k / nv
        center = np.array([4.0 * math.sin(th), 0.0, -4.0 * math.cos(th)])
        f = -center / np.linalg.norm(center)
        right = np.cross([0.0, 1.0, 0.0], f)
        right /= np.linalg.norm(right)
        R = np.stack([right, np.cross(f, right), f])
        focal = float(np.float32((w / 2.0) / math.tan(math.radians(30.0))))
        out.append(View(k % n_scenes, w, h, R.astype(np.float32),
                        (-R @ center).astype(np.float32), focal, focal, w / 2.0, h / 2.0,
                        float(np.float32(k / (nv - 1) if nv > 1 else time0)),
                        tuple(float(np.float32(x)) for x in rng.uniform(0.2, 0.8, size=3))))
    return out


def _pixels(views):
    return sum(v.width * v.height for v in views)


def _smooth_images(views, g, noise):
    """Smooth images in [0, 1] with a little noise, as photographs are to a window of 11."""
    out = []
    for v in views:
        small = torch.rand((1, 3, 9, 13), generator=g, device="cuda")
        big = torch.nn.functional.interpolate(small, size=(v.height, v.width), mode="bilinear")
        big = big + noise * torch.randn(big.shape, generator=g, device="cuda")
        out.append(big[0].permute(1, 2, 0).reshape(-1, 3))
    return torch.cat(out).clamp_(0.0, 1.0).contiguous()


def _inputs(case, seed):
    """The tensors of a case."""
    kind, g = case["kind"], _gen(seed)
    if kind == "ssim":
        views = _views(case, seed)
        target = _smooth_images(views, g, 0.02)
        image = (target + 0.1 * torch.randn(target.shape, generator=g, device="cuda")).clamp_(0.0, 1.0)
        return {"views": views, "image": image, "target": target}
    if kind in ("adam", "relocate"):
        dim, rot, n = int(case["dim"]), int(case["rot"]), int(case["n"])
        params = _scene(dim, rot, n, g)
        d = {"params": params,
             "m": torch.randn(params.shape, generator=g, device="cuda") * 1e-4,
             "v": torch.rand(params.shape, generator=g, device="cuda") * 1e-6 + 1e-9}
        if kind == "adam":
            d["dparams"] = torch.randn(params.shape, generator=g, device="cuda") * 1e-3
            d["noise"] = (torch.randn((3, n), generator=g, device="cuda") * 1e-4
                          if case["noise"] else None)
        else:
            row = _rows(dim, rot)[0]["o"]
            dead = torch.rand(n, generator=g, device="cuda") < float(case["dead"])
            o = params[row].clamp(min=0.006)
            d["opacity"] = torch.where(dead, torch.rand(n, generator=g, device="cuda") * 0.0049, o)
            d["uniforms"] = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
        return d
    views = _views(case, seed)
    sizes = [int(x) for x in case["sizes"].split(",")]
    d = {"views": views,
         "params": [_scene(int(case["dim"]), int(case["rot"]), n, _gen(seed, 1 + k))
                    for k, n in enumerate(sizes)]}
    if kind in ("frame", "replay"):
        d["target"] = torch.rand((_pixels(views), 3), generator=g, device="cuda")
    elif kind == "train":
        d["target"] = _smooth_images(views, g, 0.02)
    elif kind == "render":
        A = _pixels(views)
        d["d_image"] = torch.randn((A, 3), generator=g, device="cuda") / (3 * A)
        d["d_t"] = torch.randn((A,), generator=g, device="cuda") / A
    return d


def prepare(case, seed):
    s = dict(_inputs(case, seed), kind=case["kind"], case=case)
    kind = s["kind"]
    if kind in FRAMES:
        dim, rot = int(case["dim"]), int(case["rot"])
        s["renderer"] = ubs.Renderer(ubs.Tuning(flags=ubs.UBS_TUNE_PRE_FP32 if case["fp32"] else 0))
        s["dims"], s["rots"] = [dim] * len(s["params"]), [rot] * len(s["params"])
        if kind == "render":
            s["params"] = [p.requires_grad_(True) for p in s["params"]]
        s["scenes"] = [ubs.SceneRef(p.detach(), dim, rot) for p in s["params"]]
        if kind == "replay":
            s["graph"] = GraphFrame(s["renderer"], s["scenes"], s["views"], l1_target=s["target"])
    return s


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "view":
        return s["renderer"].forward(s["scenes"], s["views"])
    if kind == "frame":
        image, t = s["renderer"].forward(s["scenes"], s["views"])
        return image, t, s["renderer"].backward(l1_image=image, l1_target=s["target"])
    if kind == "replay":
        s["graph"].replay()
        return s["graph"].image, s["graph"].t_final, s["graph"].dparams
    if kind == "render":
        image, t = ubs.render(s["renderer"], s["params"], s["dims"], s["rots"], s["views"])
        return image.detach(), t.detach(), list(torch.autograd.grad((image, t), s["params"],
                                                                    (s["d_image"], s["d_t"])))
    if kind == "train":
        image, t = s["renderer"].forward(s["scenes"], s["views"])
        loss, d_image = ubs.ssim_loss(image, s["target"], s["views"], LAMBDA_SSIM)
        return image, t, s["renderer"].backward(d_image), loss.float()   # (as a program logs it)
    if kind == "ssim":
        loss, d_image = ubs.ssim_loss(s["image"], s["target"], s["views"], LAMBDA_SSIM)
        return d_image, loss.float()
    if kind == "adam":
        ubs.adam_step(s["params"], s["dparams"], s["m"], s["v"], ADAM_STEP, int(case["dim"]),
                      int(case["rot"]), noise=s["noise"])
        return s["params"], s["m"], s["v"]
    # relocate: the opacities as the optimiser left them, the same share dead in each pass
    s["params"][_rows(int(case["dim"]), int(case["rot"]))[0]["o"]].copy_(s["opacity"])
    targets, n_dead = ubs.relocate(s["params"], s["m"], s["v"], s["uniforms"], int(case["dim"]),
                                   int(case["rot"]), O_MIN)
    return s["params"], s["m"], s["v"], targets, n_dead


def work(case):
    kind = case["kind"]
    if kind == "ssim":
        A = _pixels(_views(case, 0))
        # image and target in, gradient out; two separable 11-tap windows of 4 and 3 planes a channel
        return {"bytes": 36.0 * A, "flops": 3.0 * A * 2 * 22 * 7}
    if kind in ("adam", "relocate"):
        F, n = _rows(int(case["dim"]), int(case["rot"]))[1], int(case["n"])
        if kind == "adam":   # parameters, gradient and two moments in, three of them out
            return {"bytes": 28.0 * F * n + (12.0 * n if case["noise"] else 0), "flops": 14.0 * F * n}
        d = float(case["dead"])   # every parameter in; a dead one's row taken and three rows written
        return {"bytes": 4.0 * F * n + 16.0 * F * n * d + 8.0 * F * n * d + 12.0 * n, "flops": float(n)}
    views = _views(case, 0)
    F, c = _rows(int(case["dim"]), int(case["rot"]))[1], int(case["dim"]) - 3
    sizes = [int(x) for x in case["sizes"].split(",")]
    A, n_rec, bwd = _pixels(views), sum(sizes[v.scene] for v in views), kind != "view"
    # parameters in, image and transmittance out; backward: gradient or target in, gradients out
    b = 4.0 * F * sum(sizes) + 16.0 * A
    if bwd:
        b += 4.0 * F * sum(sizes) + 12.0 * A
    # per record the query block (its products, factor, inverse) and the projection; about half
    # a tile pair a record, a third of whose 256 pixels it covers
    f = n_rec * (200.0 + 8.0 * c * c + 2.0 * c ** 3) + n_rec * 0.5 * 85.0 * (20.0 + (45.0 if bwd else 0.0))
    if kind == "train":
        b, f = b + 36.0 * A, f + 3.0 * A * 2 * 22 * 7
    return {"bytes": b, "flops": f}


# ------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    kind, d = case["kind"], _inputs(case, seed)
    if kind == "ssim":
        loss, grad = _ssim64(d["image"].double(), d["target"].double(), d["views"])
        return grad, loss
    if kind == "adam":
        return _adam64(case, d)
    if kind == "relocate":
        return _relocate64(case, d)
    return _frame64(case, d)


def _blur64(z):
    """The normalised 11-tap Gaussian window, sigma 1.5, over the last two axes, zeros outside."""
    x = torch.arange(-5, 6, dtype=torch.float64, device=z.device)
    g = torch.exp(-x * x / 4.5)
    g = (g / g.sum()).tolist()
    for ax in (-1, -2):
        n = z.shape[ax]
        pad = torch.nn.functional.pad(z, (5, 5) if ax == -1 else (0, 0, 5, 5))
        z = sum(g[k] * pad.narrow(ax, k, n) for k in range(11))
    return z


def _ssim64(image, target, views):
    n, k, loss, grads = float(image.numel()), 0, 0.0, []
    for v in views:
        m = v.width * v.height
        X, Y = (q[k:k + m].view(v.height, v.width, 3).permute(2, 0, 1) for q in (image, target))
        k += m
        X = X.detach().clone().requires_grad_(True)
        mx, my = _blur64(X), _blur64(Y)
        sx, sy, sxy = _blur64(X * X) - mx * mx, _blur64(Y * Y) - my * my, _blur64(X * Y) - mx * my
        s = ((2 * mx * my + 1e-4) * (2 * sxy + 9e-4)) / ((mx * mx + my * my + 1e-4) * (sx + sy + 9e-4))
        one = (1 - LAMBDA_SSIM) * (X - Y).abs().sum() / n - LAMBDA_SSIM * s.sum() / n
        grads.append(torch.autograd.grad(one, X)[0].permute(1, 2, 0).reshape(-1, 3))
        loss = loss + one.detach()
    return (loss + LAMBDA_SSIM).reshape(1), torch.cat(grads)


def _adam64(case, d):
    at, F = _rows(int(case["dim"]), int(case["rot"]))
    cfg = ubs.AdamConfig()
    p, g, m, v = (d[k].double() for k in ("params", "dparams", "m", "v"))
    lr = torch.full((F, 1), float(np.float32(cfg.lr_other)), dtype=torch.float64, device="cuda")
    for name, k, rate in (("mu", 3, cfg.lr_mu_x), ("logs", 3, cfg.lr_scale), ("o", 1, cfg.lr_opacity)):
        lr[at[name]:at[name] + k] = float(np.float32(rate))
    f32 = lambda x: float(np.float32(x))  # noqa: E731  the settings are float32
    b1, b2 = f32(cfg.beta1), f32(cfg.beta2)
    o, s = slice(at["o"], at["o"] + 1), slice(at["logs"], at["logs"] + 3)
    g[o] += f32(cfg.lambda_o) * torch.sign(p[o])
    g[s] += f32(cfg.lambda_s) * torch.exp(p[s])
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    p = p - lr * (m / (1 - b1 ** ADAM_STEP)) / ((v / (1 - b2 ** ADAM_STEP)).sqrt() + f32(cfg.eps))
    if d["noise"] is not None:
        p[:3] += f32(cfg.lambda_eps) * d["noise"].double()
    return p, m, v


def _relocate64(case, d):
    row = _rows(int(case["dim"]), int(case["rot"]))[0]["o"]
    p, m, v = (d[k].double() for k in ("params", "m", "v"))
    p[row] = d["opacity"].double()
    n = p.shape[1]
    dead = d["opacity"] < np.float32(O_MIN)
    cdf = torch.cumsum(torch.where(dead, torch.zeros_like(p[row]), p[row]), 0)
    idx = torch.nonzero(dead).view(-1)
    pick = torch.searchsorted(cdf, d["uniforms"][:idx.numel()] * cdf[-1], right=True)
    copies = torch.bincount(pick, minlength=n)
    o = torch.where(copies > 0, 1 - (1 - p[row]) ** (1.0 / (copies.double() + 1)), p[row])
    p[:, idx] = p[:, pick]
    o[idx] = o[pick]
    p[row] = o
    moved = dead | (copies > 0)
    m[:, moved] = 0
    v[:, moved] = 0
    targets = torch.zeros(n, dtype=torch.int32, device="cuda")
    targets[:idx.numel()] = pick.to(torch.int32)
    return p, m, v, targets, torch.tensor([idx.numel()], device="cuda")


def _records64(P, dim, rot, view):
    """Screen-space records of the columns of P (float64 [F][m]) in one view: a dict of [m]
    tensors, with `live`."""
    at, _ = _rows(dim, rot)
    c = dim - 3
    R = [[float(x) for x in r] for r in np.asarray(view.R, dtype=np.float64)]
    tr = [float(x) for x in np.asarray(view.t, dtype=np.float64)]
    cam = [float(np.float32(-sum(R[j][k] * tr[j] for j in range(3)))) for k in range(3)]
    q = [P[at["rot"] + k] for k in range(4 if rot == QUAT else 3)]
    one = torch.ones_like(P[0])
    if rot == QUAT:
        inv = 1.0 / (q[0] ** 2 + q[1] ** 2 + q[2] ** 2 + q[3] ** 2).sqrt()
        w, x, y, z = (k * inv for k in q)
        Q = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
             [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
             [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    else:
        Q = [[one, -q[2], q[1]], [q[2], one, -q[0]], [-q[1], q[0], one]]
    s = [P[at["logs"] + k].exp() for k in range(3)]
    M = [[Q[a][b] * s[b] for b in range(3)] for a in range(3)]
    S = [[sum(M[a][k] * M[b][k] for k in range(3)) for b in range(3)] for a in range(3)]
    mu = [P[at["mu"] + k] for k in range(3)]
    oq = P[at["o"]]
    if c:
        dv = [mu[k] - cam[k] for k in range(3)]
        dist = (dv[0] ** 2 + dv[1] ** 2 + dv[2] ** 2).sqrt()
        dirs = [k / dist for k in dv]
        query = dirs if c == 3 else [view.time * one] + dirs + [view.query[k] * one for k in range(c - 4)]
        v = [query[k] - P[at["muq"] + k] for k in range(c)]
        Lx = [[P[at["lqx"] + 3 * a + b] for b in range(3)] for a in range(c)]
        L, k = [[None] * c for _ in range(c)], at["lq"]
        for i in range(c):
            for j in range(i + 1):
                L[i][j] = P[k].exp() if i == j else P[k]
                k += 1
        H = [[None] * c for _ in range(c)]     # Cholesky factor of the query block
        for j in range(c):
            for i in range(j, c):
                a = sum(Lx[i][k] * Lx[j][k] for k in range(3)) + sum(L[i][k] * L[j][k] for k in range(j + 1))
                for k in range(j):
                    a = a - H[i][k] * H[j][k]
                H[i][j] = a.sqrt() if i == j else a / H[j][j]

        def solve(b):                          # H^-1 b
            y = []
            for i in range(c):
                a = b[i]
                for k in range(i):
                    a = a - H[i][k] * y[k]
                y.append(a / H[i][i])
            return y

        def solve_t(b):                        # H^-T b
            y = [None] * c
            for i in reversed(range(c)):
                a = b[i]
                for k in range(i + 1, c):
                    a = a - H[k][i] * y[k]
                y[i] = a / H[i][i]
            return y

        wv = solve(v)
        bq = [P[at["bq"] + k].exp() for k in range(c)]
        # log(1 - tanh x) = log 2 - 2 x - log(1 + exp(-2 x)) at x = w^2
        oq = oq * sum(4 * bq[k] * (math.log(2.0) - 2 * wv[k] ** 2 - torch.log1p(torch.exp(-2 * wv[k] ** 2)))
                      for k in range(c)).exp()
        bt = [k.clamp(max=1.0) for k in bq]
        X = [[sum(M[a][k] * Lx[j][k] for k in range(3)) for j in range(c)] for a in range(3)]
        K = [solve_t(solve(X[a])) for a in range(3)]
        mu = [mu[a] + sum(K[a][k] * bt[k] * v[k] for k in range(c)) for a in range(3)]
        S = [[S[a][b] - 0.5 * sum(bt[k] * (K[a][k] * X[b][k] + K[b][k] * X[a][k]) for k in range(c))
              for b in range(3)] for a in range(3)]
    p = [sum(R[a][k] * mu[k] for k in range(3)) + tr[a] for a in range(3)]
    z = torch.where(p[2] > NEAR, p[2], one)
    J = [[view.fx / z, None, -view.fx * p[0] / z ** 2], [None, view.fy / z, -view.fy * p[1] / z ** 2]]
    T = [[J[0][0] * R[0][b] + J[0][2] * R[2][b] for b in range(3)],
         [J[1][1] * R[1][b] + J[1][2] * R[2][b] for b in range(3)]]
    TS = [[sum(T[a][k] * S[k][b] for k in range(3)) for b in range(3)] for a in range(2)]
    s00 = sum(TS[0][k] * T[0][k] for k in range(3)) + DILATION
    s01 = sum(TS[0][k] * T[1][k] for k in range(3))
    s11 = sum(TS[1][k] * T[1][k] for k in range(3)) + DILATION
    det = s00 * s11 - s01 * s01
    beta = 4 * P[at["bx"]].exp()
    live = (p[2] > NEAR) & (det > 0) & (s00 > 0) & (s11 > 0) & (oq >= ALPHA_MIN)
    rho = torch.where(oq >= ALPHA_MIN, 1 - (255.0 * oq.clamp(min=ALPHA_MIN)) ** (-1.0 / beta), -one)
    det = torch.where(det > 0, det, one)
    return {"live": live & (rho > 0), "mx": view.fx * p[0] / z + view.cx, "my": view.fy * p[1] / z + view.cy,
            "a": s11 / det, "b": -s01 / det, "c": s00 / det, "rho": rho, "o": oq, "beta": beta,
            "r": P[at["rgb"]], "g": P[at["rgb"] + 1], "bl": P[at["rgb"] + 2], "z": p[2]}


FIELDS = ("mx", "my", "a", "b", "c", "o", "beta", "r", "g", "bl")
COLUMNS, CELLS = 400_000, 24_000_000


def _live64(P32, dim, rot, view):
    """Indices, differentiable fields [10][m], rho and depth of the live records of one view."""
    parts = []
    for k in range(0, P32.shape[1], COLUMNS):
        r = _records64(P32[:, k:k + COLUMNS].double(), dim, rot, view)
        i = torch.nonzero(r["live"]).view(-1)
        parts.append((i + k, torch.stack([r[f][i] for f in FIELDS]), r["rho"][i], r["z"][i]))
    return tuple(torch.cat([p[q] for p in parts], dim=-1) for q in range(4))


def _raster64(rec, rho, depth, view, grad_of):
    """Composites one view in 16 x 16 tiles.  grad_of(pixel indices, colour, T) gives the gradients of both (or None);
    returns image, T and the gradient of rec."""
    W, H = view.width, view.height
    tx, ty = (W + 15) // 16, (H + 15) // 16
    dev = rec.device
    image = torch.zeros((H * W, 3), dtype=torch.float64, device=dev)
    final = torch.ones(H * W, dtype=torch.float64, device=dev)
    g_rec = torch.zeros_like(rec)
    mx, my, a, b, c = rec[:5]
    det = a * c - b * b
    ex, ey = (rho * c / det).sqrt() + 1.0, (rho * a / det).sqrt() + 1.0
    x0, x1 = ((mx - ex) / 16).floor().clamp(0, tx), ((mx + ex) / 16).floor().clamp(-1, tx - 1)
    y0, y1 = ((my - ey) / 16).floor().clamp(0, ty), ((my + ey) / 16).floor().clamp(-1, ty - 1)
    nx, ny = (x1 - x0 + 1).clamp(min=0).long(), (y1 - y0 + 1).clamp(min=0).long()
    order = torch.argsort(depth, stable=True)
    cnt = (nx * ny)[order]
    who = torch.repeat_interleave(order, cnt)
    k = torch.arange(who.numel(), device=dev) - torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
    wide = nx[who].clamp(min=1)
    tile = (y0.long()[who] + k // wide) * tx + x0.long()[who] + k % wide
    tile, by = torch.sort(tile, stable=True)      # depth order is kept inside a tile
    who = who[by]
    count = torch.bincount(tile, minlength=tx * ty)
    start = count.cumsum(0) - count
    tiles = torch.argsort(count, descending=True)
    lengths = count[tiles].tolist()
    at = 0
    while at < len(lengths) and lengths[at] > 0:
        deep = lengths[at]
        some = tiles[at:at + max(1, CELLS // (256 * deep))]
        at += some.numel()
        slot = torch.arange(deep, device=dev)
        have = slot[None, :] < count[some][:, None]
        idx = who[(start[some][:, None] + slot[None, :]).clamp(max=who.numel() - 1)]
        px = (some % tx)[:, None] * 16 + torch.arange(256, device=dev)[None, :] % 16
        py = (some // tx)[:, None] * 16 + torch.arange(256, device=dev)[None, :] // 16
        inside = (px < W) & (py < H)
        pix = (py * W + px)[inside]
        sub = rec[:, idx].detach().requires_grad_(grad_of is not None)
        with torch.set_grad_enabled(grad_of is not None):
            f = [q[:, :, None] for q in sub]
            dx, dy = px[:, None, :] + 0.5 - f[0], py[:, None, :] + 0.5 - f[1]
            r = f[2] * dx * dx + 2 * f[3] * dx * dy + f[4] * dy * dy
            on = have[:, :, None] & (r <= rho[idx][:, :, None])
            sigma = f[5] * (1 - torch.where(on, r, torch.zeros_like(r))) ** f[6]
            on = on & (sigma >= ALPHA_MIN)
            alpha = torch.where(on, sigma.clamp(max=ALPHA_MAX), torch.zeros_like(r))
            alpha = alpha * (torch.cumprod(1 - alpha, 1) >= T_STOP)
            T = torch.cumprod(1 - alpha, 1)
            w = alpha * torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
            col = torch.stack([(w * f[7 + q]).sum(1) for q in range(3)], -1)
            tf = T[:, -1]
        image[pix], final[pix] = col.detach()[inside], tf.detach()[inside]
        if grad_of is not None:
            gi, gt = grad_of(pix, image[pix], final[pix])
            g1 = torch.zeros_like(col)
            g1[inside] = gi
            out, grads = [col], [g1]
            if gt is not None:
                g2 = torch.zeros_like(tf)
                g2[inside] = gt
                out, grads = out + [tf], grads + [g2]
            g = torch.autograd.grad(out, sub, grads)[0]
            g_rec.index_add_(1, idx[have], g[:, have])
    return image, final, g_rec


def _frame64(case, d):
    kind, dim, rot, views = case["kind"], int(case["dim"]), int(case["rot"]), d["views"]
    A, bwd = _pixels(views), kind != "view"
    images, finals, base = [], [], 0
    grads = [torch.zeros(p.shape, dtype=torch.float64, device="cuda") for p in d["params"]] if bwd else None
    loss = given = None
    if kind == "train":   # the loss needs the whole image first
        for v in views:
            rec = _live64(d["params"][v.scene], dim, rot, v)
            images.append(_raster64(*rec[1:], v, None)[0])
        loss, given = _ssim64(torch.cat(images), d["target"].double(), views)
        images = []
    for v in views:
        lo, P32 = base, d["params"][v.scene]
        base += v.width * v.height

        def grad_of(pix, col, tf):
            if kind == "render":
                return d["d_image"][lo + pix].double(), d["d_t"][lo + pix].double()
            if kind == "train":
                return given[lo + pix], None
            return torch.sign(col - d["target"][lo + pix].double()) / (3.0 * A), None

        i, rec, rho, depth = _live64(P32, dim, rot, v)
        image, final, g_rec = _raster64(rec, rho, depth, v, grad_of if bwd else None)
        images.append(image)
        finals.append(final)
        for k in range(0, i.numel() if bwd else 0, COLUMNS):
            some = i[k:k + COLUMNS]
            P = P32[:, some].double().requires_grad_(True)
            r = _records64(P, dim, rot, v)
            out = torch.stack([r[f] for f in FIELDS])
            grads[v.scene].index_add_(1, some, torch.autograd.grad(out, P, g_rec[:, k:k + COLUMNS])[0])
    out = [torch.cat(images), torch.cat(finals)]
    if bwd:
        out.append(grads)
    if kind == "train":
        out.append(loss)
    return out
