"""Timed cases of fourth-order EED inpainting with FSI: what a program that uses
this package has it do, through the public entry points.

A case is a dict of plain values.  Its "kind" names the entry point:
  inpaint  eed4_inpaint of B equal-size images, a fixed number of cycles or
           until the relative residual is below tol
  step     eed4_fsi_step, one inner step
  batch    eed4_inpaint_batched of images of uneven sizes
  train    one tonal-optimisation step through the autograd wrapper: forward,
           mean squared error, gradient with respect to the known values
Images are piecewise smooth (ellipses over a ramp, with noise) with a few
percent of the pixels known, as in the repository's workloads; the unknown
pixels start at the mean of the known ones.
"""
import math

import numpy as np
import torch

import paper_2006_10406_amd as eed4
from paper_2006_10406_amd import autograd as eed4_autograd

DEV = "cuda"
MAX_R = 8
SIDES = (128, 1024)            # sides of the images of an uneven batch


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "B": 1, "H": 0, "W": 0, "sigma": 1.5, "lam": 0.03,
         "tau": 0.05, "n": 15, "M": 1, "tol": 0.0, "diff": 0, "mu3": 0, "density": 0.04,
         "ellipses": 30, "noise": 0.01}
    c.update(kw)
    return c


def listed():
    return [
        # a thumbnail to the end of its run: launches and latency are all of it
        _case("small64", "inpaint", H=64, W=64, sigma=1.0, lam=0.05, n=10, M=20, density=0.05,
              ellipses=5),
        # one photograph-sized image to the stop rule, one residual read per cycle of 40
        _case("single512_to_tol", "inpaint", H=512, W=512, n=40, M=400, tol=1e-4),
        # colour: three planes that share their mask, a fixed number of cycles
        _case("rgb512", "inpaint", B=3, H=512, W=512, M=40, density=0.05),
        # odd sizes, the widest presmoothing
        _case("ragged1037x771", "inpaint", H=1037, W=771, sigma=2.6, n=15, M=8),
        # odd sizes, hardly any presmoothing (no odd side is a multiple of anything)
        _case("ragged613x1999", "inpaint", H=613, W=1999, sigma=0.5, lam=0.05, n=20, M=6),
        # a scan at full size: the repository's headline workload, ten of its cycles
        _case("large4096", "inpaint", H=4096, W=4096, sigma=2.0, lam=0.02, n=15, M=10,
              density=0.03, noise=0.005, ellipses=60),
        # a single step on an image beyond every cache
        _case("step8192", "step", H=8192, W=8192, sigma=2.0, lam=0.02, n=15, density=0.03,
              noise=0.005, ellipses=60),
        # a tensor variant (exponential Perona-Malik, arithmetic-mean mu3)
        _case("variant2048", "inpaint", H=2048, W=2048, sigma=2.0, lam=0.02, n=15, M=8, diff=2,
              mu3=1),
        # a folder of images of all sizes in one call
        _case("batch64", "batch", B=64, H=SIDES[0], W=SIDES[1], M=10, density=0.05, noise=0.005),
        # tonal optimisation: one training step on a stack of small images ...
        _case("train16x256", "train", B=16, H=256, W=256, sigma=1.0, lam=0.05, n=10, M=30),
        # ... and on one large image
        _case("train2048", "train", H=2048, W=2048, sigma=2.0, lam=0.02, n=15, M=2, density=0.03),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["inpaint", "inpaint", "inpaint", "step", "batch", "train"])
    c = _case("", kind, sigma=round(rng.uniform(0.3, 2.66), 2) if rng.random() < 0.9 else 0.0,
              lam=round(rng.uniform(0.02, 0.06), 4), tau=rng.choice([0.05, 0.05, 0.06]),
              n=rng.randint(8, 40), density=round(rng.uniform(0.02, 0.1), 3),
              noise=rng.choice([0.005, 0.01]))
    if kind == "inpaint":
        c["H"], c["W"] = _loguniform(rng, 48, 4096), _loguniform(rng, 48, 4096)
        px = c["H"] * c["W"]
        if px < 1 << 18:
            c["B"] = rng.choice([1, 1, 3, 8])
        # at most the updates of the largest listed run
        c["M"] = max(1, min(rng.randint(4, 40), int(1.2e9 / (px * c["B"] * c["n"]))))
        if rng.random() < 0.25:
            c["diff"], c["mu3"] = rng.randint(0, 3), rng.randint(0, 2)
    elif kind == "step":
        c["H"], c["W"] = _loguniform(rng, 512, 8192), _loguniform(rng, 512, 8192)
    elif kind == "batch":
        c["B"], c["H"], c["W"] = rng.randint(4, 64), SIDES[0], rng.randint(300, SIDES[1])
        c["n"], c["M"] = rng.randint(8, 20), rng.randint(3, 10)
    else:
        side = (64, 1024)
        c["H"], c["W"] = _loguniform(rng, *side), _loguniform(rng, *side)
        c["B"] = max(1, min(16, (1 << 20) // (c["H"] * c["W"])))
        c["n"] = rng.randint(5, 15)
        c["M"] = max(1, min(rng.randint(2, 30), int(1.5e8 / (c["H"] * c["W"] * c["B"] * c["n"]))))
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _image(H, W, c, rng, gen):
    """One piecewise-smooth image in [0, 1], float32 on the GPU."""
    img = torch.full((H, W), float(rng.uniform()), device=DEV)
    m = min(H, W)
    for _ in range(c["ellipses"]):
        cy, cx = rng.uniform(0, H), rng.uniform(0, W)
        a, b = rng.uniform(0.05, 0.3, 2) * m
        th, grey, rad = rng.uniform(0, math.pi), float(rng.uniform()), max(a, b)
        y0, y1 = max(0, int(cy - rad)), min(H, int(cy + rad) + 2)
        x0, x1 = max(0, int(cx - rad)), min(W, int(cx + rad) + 2)
        yy = torch.arange(y0, y1, device=DEV, dtype=torch.float32)[:, None] - cy
        xx = torch.arange(x0, x1, device=DEV, dtype=torch.float32)[None, :] - cx
        p = (xx * math.cos(th) + yy * math.sin(th)) / a
        q = (yy * math.cos(th) - xx * math.sin(th)) / b
        img[y0:y1, x0:x1].masked_fill_(p * p + q * q <= 1.0, grey)
    img = 0.75 * img + 0.25 * torch.linspace(0, 1, W, device=DEV)[None, :]
    img += c["noise"] * torch.randn(img.shape, generator=gen, device=DEV)
    return img.clamp_(0.0, 1.0)


def _problem(H, W, c, rng, gen, mask=None):
    img = _image(H, W, c, rng, gen)
    if mask is None:
        mask = (torch.rand((H, W), generator=gen, device=DEV) < c["density"]).to(torch.uint8)
        mask[H // 2, W // 2] = 1
    known = img * mask
    u0 = torch.where(mask != 0, img, (known.double().sum() / mask.sum()).float())
    return {"image": img, "mask": mask, "known": known, "u0": u0}


def _sides(c):
    """The image sizes of an uneven batch: the case's own, only the images come from the seed."""
    return np.random.default_rng(c["B"]).integers(c["H"], c["W"] + 1, size=(c["B"], 2))


def _problems(c, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    if c["kind"] == "batch":
        return [_problem(int(h), int(w), c, rng, gen) for h, w in _sides(c)]
    out = []
    for b in range(c["B"]):
        # the planes of a colour image share one mask
        shared = out[0]["mask"] if c["B"] == 3 and out else None
        out.append(_problem(c["H"], c["W"], c, rng, gen, shared))
    return out


def _stack(probs, key):
    return torch.stack([p[key] for p in probs])


def _mid_run(probs):
    """u^k and u^{k-1} as in mid-run: near the image and near each other."""
    img, u0, m = _stack(probs, "image"), _stack(probs, "u0"), _stack(probs, "mask") != 0
    u = torch.where(m, img, 0.5 * (img + u0))
    return u, torch.where(m, img, 0.45 * img + 0.55 * u)


def _params(c):
    flags = eed4.EED4_DIFFUSIVITY(c["diff"]) | eed4.EED4_MU3(c["mu3"])
    return eed4.params(c["lam"], c["sigma"], c["tau"], c["n"], c["M"], tol=c["tol"], flags=flags)


def prepare(case, seed):
    c = case
    probs = _problems(c, seed)
    p = _params(c)
    s = {"case": c, "p": p}
    if c["kind"] == "batch":
        s["u0"] = [q["u0"] for q in probs]
        s["u"] = [torch.empty_like(x) for x in s["u0"]]
        s["images"] = [(u, q["mask"], q["known"], c["lam"]) for u, q in zip(s["u"], probs)]
        need = eed4.eed4_batched_workspace_size(s["images"], p)
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        return s
    for k in ("mask", "known", "u0"):
        s[k] = _stack(probs, k)
    if c["kind"] == "inpaint":
        s["u"] = torch.empty_like(s["u0"])
        need = eed4.eed4_workspace_size(eed4.EED4_OP_INPAINT, c["B"], c["H"], c["W"], p)
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    elif c["kind"] == "step":
        s["u0"], s["uprev"] = _mid_run(probs)
        s["out"] = torch.empty_like(s["u0"])
    else:
        s["image"] = _stack(probs, "image")
        s["known"].requires_grad_(True)
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "inpaint":
        s["u"].copy_(s["u0"])
        st, _ = eed4.eed4_inpaint(s["u"], s["mask"], s["known"], s["p"], ws=s["ws"])
        return {"u": s["u"], "cycles": int(st.cycles)}
    if c["kind"] == "step":
        eed4.eed4_fsi_step(s["u0"], s["uprev"], s["out"], s["mask"], s["p"], _step_index(c))
        return s["out"]
    if c["kind"] == "batch":
        torch._foreach_copy_(s["u"], s["u0"])
        eed4.eed4_inpaint_batched(s["images"], s["p"], ws=s["ws"])
        return s["u"]
    u = eed4_autograd.inpaint(s["known"], c["lam"], s["mask"], c["sigma"], c["tau"], c["n"], c["M"])
    loss = torch.mean((u - s["image"]) ** 2)
    grad, = torch.autograd.grad(loss, [s["known"]])
    return {"u": u.detach(), "grad_known": grad}


def _step_index(c):
    return c["n"] // 2


# ---------------------------------------------------------------- what a pass cannot do without

def _radius(c):
    return math.ceil(3.0 * float(np.float32(c["sigma"])))


def _pixels(c):
    if c["kind"] == "batch":
        return int(_sides(c).prod(axis=1).sum())
    return c["B"] * c["H"] * c["W"]


def work(case):
    """Each step reads u^k, u^{k-1} and the mask and writes u^{k+1} (13 bytes a pixel); a reverse
    step reads u^k, two adjoint states and the mask and writes two (21 bytes), after a second
    forward step from the cycle's checkpoint.  Flops: separable blur, tensor, stencils."""
    c = case
    steps = 1 if c["kind"] == "step" else c["n"] * c["M"]
    if c["tol"] > 0.0:
        steps = c["n"] * 34          # about where the stop rule ends such a run
    f = 4 * (2 * _radius(c) + 1) + 70
    px = _pixels(c) * steps
    if c["kind"] == "train":
        return {"bytes": px * (13 + 13 + 21), "flops": px * (3 * f + 80)}
    return {"bytes": px * 13, "flops": px * f}


# ---------------------------------------------------------------- the same in 64 bits, by torch

def _mirror(n, r):
    i = np.arange(-r, n + r) % (2 * n)
    return torch.from_numpy(np.where(i < n, i, 2 * n - 1 - i)).to(DEV)


class _Exact:
    """The FSI evolution in float64 on the mirror-extended image."""

    def __init__(self, c, H, W, mask):
        self.c, self.H, self.W, self.known = c, H, W, mask != 0
        self.R = _radius(c)
        s = float(np.float32(c["sigma"]))
        j = np.arange(-self.R, self.R + 1)
        w = np.exp(-j * j / (2.0 * s * s)) if self.R else np.ones(1)
        self.w = (w / w.sum()).tolist()
        self.il2 = 1.0 / float(np.float32(c["lam"])) ** 2
        self.tau = float(np.float32(c["tau"]))
        self.iy, self.ix = _mirror(H, self.R + 2), _mirror(W, self.R + 2)

    def mu(self, x):
        d, r = self.c["diff"], self.c["mu3"]
        g = ((1 + x) ** -0.5, 1 / (1 + x), torch.exp(-x), (1 + x) ** -2.0)[d]
        return g, (torch.sqrt(g), 0.5 * (1 + g), torch.ones_like(g))[r]

    def operator(self, u):
        R, H, W = self.R, self.H, self.W
        e = u[..., self.iy, :][..., self.ix]                       # halo R + 2
        v = sum(self.w[j] * e[..., j:j + W + 4] for j in range(2 * R + 1))
        v = sum(self.w[j] * v[..., j:j + H + 4, :] for j in range(2 * R + 1))  # halo 2
        gx = 0.5 * (v[..., 1:-1, 2:] - v[..., 1:-1, :-2])          # halo 1
        gy = 0.5 * (v[..., 2:, 1:-1] - v[..., :-2, 1:-1])
        e = e[..., R:R + H + 4, R:R + W + 4]
        m = e[..., 1:-1, 1:-1]
        hxx = e[..., 1:-1, 2:] - 2 * m + e[..., 1:-1, :-2]
        hyy = e[..., 2:, 1:-1] - 2 * m + e[..., :-2, 1:-1]
        hxy = 0.25 * (e[..., 2:, 2:] + e[..., :-2, :-2] - e[..., 2:, :-2] - e[..., :-2, 2:])
        a, b, ab = gx * gx, gy * gy, gx * gy
        s2 = a + b
        mu1, mu3 = self.mu(s2 * self.il2)
        q = 1.0 / torch.where(s2 > 1e-200, s2, torch.ones_like(s2))   # G = 0: the terms vanish
        k1 = (mu1 - 1) * (a * hxx + b * hyy + 2 * ab * hxy) * q * q
        k3 = (mu3 - 1) * (ab * (hyy - hxx) + (a - b) * hxy) * q * q
        txx = hxx + k1 * a - 2 * k3 * ab
        tyy = hyy + k1 * b + 2 * k3 * ab
        txy = hxy + k1 * ab + k3 * (a - b)
        return (txx[..., 1:-1, 2:] - 2 * txx[..., 1:-1, 1:-1] + txx[..., 1:-1, :-2]
                + tyy[..., 2:, 1:-1] - 2 * tyy[..., 1:-1, 1:-1] + tyy[..., :-2, 1:-1]
                + 0.5 * (txy[..., 2:, 2:] + txy[..., :-2, :-2] - txy[..., 2:, :-2] - txy[..., :-2, 2:]))

    def step(self, u, prev, k):
        al = (4.0 * k + 2.0) / (2.0 * k + 3.0)
        un = al * (u - self.tau * self.operator(u)) + (1.0 - al) * prev
        return torch.where(self.known, u, un)

    def cycle(self, u0):
        prev, u = u0, u0
        for k in range(self.c["n"]):
            prev, u = u, self.step(u, prev, k)
        return u


def exact(case, seed):
    c = case
    steps = 1 if c["kind"] == "step" else c["n"] * (34 if c["tol"] > 0 else c["M"])
    launches = steps * (c["B"] if c["kind"] == "batch" else 1) * (6 if c["kind"] == "train" else 1)
    if launches * 1e-3 + steps * _pixels(c) * (3e-9 if c["kind"] == "train" else 1e-9) > 20.0:
        return None
    probs = _problems(c, seed)
    with torch.no_grad():
        if c["kind"] == "batch":
            out = []
            for q in probs:
                ex = _Exact(c, *q["u0"].shape, q["mask"])
                u = q["u0"].double()
                for _ in range(c["M"]):
                    u = ex.cycle(u)
                out.append(u)
            return out
        mask = _stack(probs, "mask")
        ex = _Exact(c, c["H"], c["W"], mask)
        if c["kind"] == "step":
            u, uprev = _mid_run(probs)
            return ex.step(u.double(), uprev.double(), _step_index(c))
        if c["kind"] == "inpaint":
            u, m = _stack(probs, "u0").double(), 0
            while m < c["M"]:
                v = ex.cycle(u)
                m += 1
                dims = (-2, -1)
                rel = ((v - u).square().sum(dims).sqrt() / v.square().sum(dims).sqrt()).max()
                u = v
                if c["tol"] > 0 and float(rel) < float(np.float32(c["tol"])):
                    break
            return {"u": u, "cycles": m}
    # the training step: plain reverse-mode differentiation, cycle by cycle
    from torch.utils.checkpoint import checkpoint
    known = _stack(probs, "known").double().requires_grad_(True)
    m = (mask != 0).double()
    mean = (known * m).sum((-2, -1), keepdim=True) / m.sum((-2, -1), keepdim=True)
    u = m * known + (1.0 - m) * mean
    for _ in range(c["M"]):
        u = checkpoint(ex.cycle, u, use_reentrant=False)
    loss = torch.mean((u - _stack(probs, "image").double()) ** 2)
    grad, = torch.autograd.grad(loss, [known])
    return {"u": u.detach(), "grad_known": grad}
