"""Parity of the HIP adjoint (eed4_backward) with the FP64 oracle adjoint, a
directional finite-difference check, and tonal optimisation through the
torch.autograd wrapper.

Both adjoints differentiate the same trajectory: the oracle recomputes each
cycle in FP64 from the checkpoints the GPU forward wrote.  Bar: relative L2
<= 1e-4 and every element within 1e-4 of the largest oracle value, for dL/df
on the mask, dL/du_init off the mask, and dL/dlambda.
"""
import numpy as np
import pytest

import oracle
from synth import WORKLOADS, make_batch, make_problem
from tests.helpers import announce, assert_grad_parity, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
import paper_2006_10406_amd as eed4  # noqa: E402
from paper_2006_10406_amd import autograd as ea  # noqa: E402


def gpu_forward_backward(b, lam, sigma, tau, n, M, gu, flags=0):
    u = to_dev(b["u_init"])
    mask, known = to_dev(b["mask"]), to_dev(b["known"])
    B, H, W = u.shape
    p = eed4.params(lam, sigma, tau, n, M, flags=flags)
    ck = torch.empty((M, B, H, W), dtype=torch.float32, device="cuda")
    eed4.eed4_inpaint(u, mask, known, p, ckpt=ck)
    g = to_dev(gu.astype(np.float32))
    gk, gi = torch.empty_like(g), torch.empty_like(g)
    gl = torch.empty(B, device="cuda")
    eed4.eed4_backward(ck, mask, known, p, M, g, gk, gi, gl)
    torch.cuda.synchronize()
    return (u.cpu().numpy(), ck.cpu().numpy(), gk.cpu().numpy(), gi.cpu().numpy(),
            gl.cpu().numpy())


def compare(b, ck, gk, gi, gl, lam, sigma, tau, n, gu, label):
    ogk, ogi, ogl = oracle.backward(ck.astype(np.float64), b["mask"], b["known"], lam, sigma, tau,
                                    n, gu)
    m = b["mask"] != 0
    print(f"{label}: dL/dlambda gpu {gl[:2]}, oracle {np.atleast_1d(ogl)[:2]}")
    assert np.all(gk[~m] == 0) and np.all(gi[m] == 0)
    assert_grad_parity(gk[m], ogk[m], f"{label} dL/df")
    assert_grad_parity(gi[~m], ogi[~m], f"{label} dL/du_init")
    assert_grad_parity(gl, ogl, f"{label} dL/dlambda")


@pytest.mark.parametrize("H,W,sigma,lam,n,M", [
    (40, 52, 1.0, 0.05, 5, 3), (67, 45, 1.5, 0.03, 4, 2), (33, 70, 2.0, 0.02, 3, 2),
    (20, 17, 0.0, 0.1, 6, 2), (9, 130, 2.6, 0.05, 2, 2), (70, 66, 0.5, 0.04, 1, 3),
    # many cycles: the recompute alternates its two buffer sets across odd and even counts
    (30, 41, 1.0, 0.05, 3, 19), (26, 33, 1.5, 0.03, 2, 8)])
def test_adjoint_matches_oracle(H, W, sigma, lam, n, M):
    announce(f"adjoint {H}x{W} sigma={sigma} n={n} M={M}")
    b = {k: np.stack([make_problem(H, W, 4, True, 0.01, 0.08, 900 + i + H)[k] for i in range(2)])
         for k in ("image", "mask", "known", "u_init")}
    gu = np.random.default_rng(H * W).normal(size=b["u_init"].shape) * 1e-2
    _, ck, gk, gi, gl = gpu_forward_backward(b, lam, sigma, 0.05, n, M, gu)
    compare(b, ck, gk, gi, gl, lam, sigma, 0.05, n, gu, f"{H}x{W} s{sigma} n{n}")


@pytest.mark.parametrize("shape", range(len(eed4.SHAPE_NAMES)))
@pytest.mark.parametrize("H,W,sigma,n", [(75, 140, 1.0, 4), (131, 62, 2.0, 3), (7, 200, 0.5, 2)])
def test_each_reverse_step_kernel_matches_oracle(shape, H, W, sigma, n):
    # tile shapes select the two-pass tile adjoint, strip shapes the fused
    # strip adjoint of that segment height (and the same forward shape)
    announce(f"reverse step {eed4.SHAPE_NAMES[shape]} {H}x{W} sigma={sigma} n={n}")
    b = {k: np.stack([make_problem(H, W, 5, True, 0.01, 0.06, 700 + i + W)[k] for i in range(2)])
         for k in ("image", "mask", "known", "u_init")}
    gu = np.random.default_rng(H + W).normal(size=b["u_init"].shape) * 1e-2
    _, ck, gk, gi, gl = gpu_forward_backward(b, 0.04, sigma, 0.05, n, 2, gu,
                                             flags=eed4.EED4_FORCE_SHAPE(shape))
    compare(b, ck, gk, gi, gl, 0.04, sigma, 0.05, n, gu,
            f"{eed4.SHAPE_NAMES[shape]} {H}x{W} s{sigma}")


@pytest.mark.parametrize("shape", [0, 3, 6])
@pytest.mark.parametrize("H,W", [(1, 1), (2, 3), (1, 40), (37, 1)])
def test_reverse_step_degenerate_sizes(shape, H, W):
    # one pixel, single rows and columns: every neighbour comes from the
    # mirror (repeated reflection), in both the recompute and the reverse step
    announce(f"reverse step {eed4.SHAPE_NAMES[shape]} degenerate {H}x{W}")
    b = {k: np.stack([make_problem(H, W, 2, True, 0.01, 0.25, 40 + i + 3 * H + W)[k]
                      for i in range(2)]) for k in ("image", "mask", "known", "u_init")}
    gu = np.random.default_rng(7 + H * W).normal(size=b["u_init"].shape) * 1e-2
    _, ck, gk, gi, gl = gpu_forward_backward(b, 0.05, 1.0, 0.05, 4, 2, gu,
                                             flags=eed4.EED4_FORCE_SHAPE(shape))
    compare(b, ck, gk, gi, gl, 0.05, 1.0, 0.05, 4, gu,
            f"{eed4.SHAPE_NAMES[shape]} {H}x{W}")


def test_adjoint_tile_kernel_recompute():
    announce("adjoint with the tile step kernel for the recompute")
    b = {k: v[None] for k, v in make_problem(48, 60, 4, True, 0.01, 0.06, 31).items()
         if k in ("image", "mask", "known", "u_init")}
    gu = np.random.default_rng(3).normal(size=b["u_init"].shape) * 1e-2
    _, ck, gk, gi, gl = gpu_forward_backward(b, 0.05, 1.0, 0.05, 5, 2, gu,
                                             flags=eed4.EED4_TILE_KERNEL)
    compare(b, ck, gk, gi, gl, 0.05, 1.0, 0.05, 5, gu, "tile recompute")


def test_adjoint16_workload_sampled_images():
    wl = WORKLOADS["adjoint16"]
    announce("adjoint16: 16 x 256x256, 30 cycles of 10; oracle on images 0 and 9")
    b = make_batch(wl)
    u_gpu = None
    gu = None
    # loss = MSE against the ground truth, seed 2 (u - gt) / N
    u = to_dev(b["u_init"])
    mask, known = to_dev(b["mask"]), to_dev(b["known"])
    B, H, W = u.shape
    p = eed4.params(wl.lam, wl.sigma, wl.tau, wl.n, wl.M)
    ck = torch.empty((wl.M, B, H, W), dtype=torch.float32, device="cuda")
    eed4.eed4_inpaint(u, mask, known, p, ckpt=ck)
    u_gpu = u.cpu().numpy()
    gu = 2.0 * (u_gpu - b["image"]) / u_gpu.size
    g = to_dev(gu.astype(np.float32))
    gk, gi = torch.empty_like(g), torch.empty_like(g)
    gl = torch.empty(B, device="cuda")
    eed4.eed4_backward(ck, mask, known, p, wl.M, g, gk, gi, gl)
    torch.cuda.synchronize()
    ckn, gkn, gin, gln = ck.cpu().numpy(), gk.cpu().numpy(), gi.cpu().numpy(), gl.cpu().numpy()
    for i in (0, 9):
        sub = {k: b[k][i:i + 1] for k in ("image", "mask", "known", "u_init")}
        compare(sub, ckn[:, i:i + 1], gkn[i:i + 1], gin[i:i + 1], gln[i:i + 1], wl.lam, wl.sigma,
                wl.tau, wl.n, gu[i:i + 1], f"adjoint16 image {i}")


def test_directional_finite_difference_on_gpu():
    announce("directional FD of the GPU forward vs GPU adjoint")
    pr = make_problem(64, 64, 5, True, 0.01, 0.05, 1234)
    image = to_dev(pr["image"])
    mask = to_dev(pr["mask"])
    m = mask.float()
    known = (image * m).contiguous()
    lam, sigma, tau, n, M = 0.05, 1.0, 0.05, 10, 5
    kp = known.clone().requires_grad_(True)
    u = ea.inpaint(kp, lam, mask, sigma, tau, n, M)
    loss = torch.sum((u - image) ** 2)
    loss.backward()
    g = kp.grad.detach()
    v = (torch.randn_like(known) * m).contiguous()
    h = 1e-3

    def L(k):
        with torch.no_grad():
            uu = ea.inpaint(k.contiguous(), lam, mask, sigma, tau, n, M)
            return float(torch.sum((uu.double() - image.double()) ** 2))

    fd = (L(known + h * v) - L(known - h * v)) / (2 * h)
    an = float(torch.sum(g * v))
    print(f"directional FD {fd:.6e} vs adjoint {an:.6e}")
    assert abs(fd - an) <= 1e-2 * abs(an)


def test_tonal_optimisation_decreases_mse():
    wl = WORKLOADS["adjoint16"]
    announce("tonal optimisation: 50 Adam steps on 16 x 256x256")
    b = make_batch(wl)
    image = to_dev(b["image"])
    mask = to_dev(b["mask"])
    out = ea.tonal_optimize(image, mask, wl.lam, wl.sigma, wl.tau, wl.n, wl.M, steps=50,
                            lr=5e-3)
    h = out["loss"]
    print(f"tonal optimisation MSE: {h[0]:.6f} -> {out['final_loss']:.6f}")
    assert out["final_loss"] < 0.9 * h[0]
    assert np.all(np.isfinite(h))


@pytest.mark.parametrize("sigma", [0.0, 1.0])
@pytest.mark.parametrize("flags", [eed4.EED4_FORCE_SHAPE(s) for s in (0, 1, 2, 3, 4, 5, 6)]
                         + [eed4.EED4_DIFFUSIVITY(2) | eed4.EED4_MU3(1)])
@pytest.mark.parametrize("H,W", [(37, 75), (100, 131)])
def test_reverse_step_takes_exact_differences_of_neighbours(H, W, flags, sigma):
    # r = 2^23 + k with k = 0..3: neighbours' differences are exact, their sums are not.  u is
    # constant, so D = I and q = 0, and one reverse step at tau = 1/16 has four roundings, all
    # known: the gradient must equal them bitwise.
    announce(f"reverse differences {H}x{W} flags {flags:#x} sigma={sigma}")
    k = np.random.default_rng(H + W).integers(0, 4, (2, H, W))
    r = (2.0 ** 23 + k).astype(np.float32)
    e = np.pad(k.astype(np.float64), ((0, 0), (2, 2), (2, 2)), mode="symmetric")
    xx = lambda a: a[:, 1:-1, 2:] - 2 * a[:, 1:-1, 1:-1] + a[:, 1:-1, :-2]
    yy = lambda a: a[:, 2:, 1:-1] - 2 * a[:, 1:-1, 1:-1] + a[:, :-2, 1:-1]
    xy = lambda a: 0.25 * ((a[:, 2:, 2:] - a[:, 2:, :-2]) - (a[:, :-2, 2:] - a[:, :-2, :-2]))
    pr = xx(xx(e)) + yy(yy(e)) + 2 * xy(xy(e))
    f32, f64 = np.float32, np.float64
    alpha = f32(2.0 / 3.0)
    stepped = (r.astype(f64) - pr / 16).astype(f32)                # products of float32 are
    scaled = (f64(alpha) * stepped.astype(f64)).astype(f32)        # exact in 64 bits
    back = (f64(f32(1.0) - alpha) * r.astype(f64)).astype(f32)
    want = (scaled.astype(f64) + back.astype(f64)).astype(f32)
    mask = torch.zeros((2, H, W), dtype=torch.uint8, device="cuda")
    ck = torch.full((1, 2, H, W), 0.5, device="cuda")
    gu = to_dev(r)
    g = [torch.empty_like(gu), torch.empty_like(gu), torch.empty(2, device="cuda")]
    eed4.eed4_backward(ck, mask, torch.zeros_like(gu), eed4.params(0.03, sigma, 1 / 16, 1, 1, flags=flags),
                       1, gu, *g)
    torch.cuda.synchronize()
    assert np.array_equal(g[1].cpu().numpy(), want)
    assert not g[0].any() and not g[2].any()


@pytest.mark.parametrize("sigma", [0.0, 0.3, 0.6, 1.0, 1.3, 1.6, 2.0, 2.3, 2.6])   # R = 0 .. 8
@pytest.mark.parametrize("H,W", [(15, 63), (16, 64), (17, 65), (33, 129), (48, 192), (50, 84), (5, 3)])
def test_presmoothing_at_the_edges_of_its_tiles(H, W, sigma):
    # with one step a cycle every presmoothed state comes from the 64 x 16 tiles of the blur
    announce(f"blur tiles {H}x{W} sigma={sigma}")
    b = {k: np.stack([make_problem(H, W, 4, True, 0.01, 0.06, 300 + i + H)[k] for i in range(2)])
         for k in ("image", "mask", "known", "u_init")}
    gu = np.random.default_rng(H * W).normal(size=b["u_init"].shape) * 1e-2
    _, ck, gk, gi, _ = gpu_forward_backward(b, 0.04, sigma, 0.05, 1, 2, gu,
                                            flags=eed4.EED4_FORCE_SHAPE(5))
    # dL/dlambda, one number an image, says nothing of a tile's edge, and for a random dL/du its
    # terms cancel: at 33x129, sigma 2.3, it is 1.2e-4 off whichever kernel presmooths
    ogk, ogi, _ = oracle.backward(ck.astype(np.float64), b["mask"], b["known"], 0.04, sigma, 0.05, 1,
                                  gu)
    m = b["mask"] != 0
    assert np.all(gk[~m] == 0) and np.all(gi[m] == 0)
    assert_grad_parity(gk[m], ogk[m], f"{H}x{W} s{sigma} dL/df")
    assert_grad_parity(gi[~m], ogi[~m], f"{H}x{W} s{sigma} dL/du_init")


def test_presmoothing_of_64_columns_is_one_tile_wide():
    # 64 x 2374x61 and x60 at sigma 1.3: the reverse strips are two wide in both, and the rest of the
    # backward differs by the pixels, 1.017.  Two blur tiles across add 40 us of some 200 at 61
    announce("backward of one step, 64 x 2374x61 against 64 x 2374x60")
    p = eed4.params(0.02, 1.3, 0.05, 1, 1, flags=eed4.EED4_FORCE_SHAPE(5))
    calls, best = {}, {}
    for W in (61, 60):
        u = torch.rand((64, 2374, W), device="cuda")
        mask, gu = (u < 0.05).to(torch.uint8), torch.randn_like(u)
        g = (torch.empty_like(u), torch.empty_like(u), torch.empty(64, device="cuda"))
        calls[W] = (u[None].contiguous(), mask, u.clone(), p, 1, gu, *g)
        best[W] = 1e9
    for _ in range(40):
        for W, args in calls.items():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            eed4.eed4_backward(*args)
            b.record()
            b.synchronize()
            best[W] = min(best[W], 1e3 * a.elapsed_time(b))
    print(f"61 columns {best[61]:.1f} us, 60 columns {best[60]:.1f} us")
    assert best[61] < 1.1 * best[60]
