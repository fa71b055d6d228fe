"""Shape 3 on images whose width strips of 60 columns fill better than strips of 124: bitwise the
tiles' results at the edges of its 64-row segments and 60-column strips, in single calls, in the
backward's recompute and in the batched queue; and faster than the 124-column strips there."""
import numpy as np
import pytest

from synth import make_problem
from tests.helpers import announce, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
import paper_2006_10406_amd as eed4  # noqa: E402

SIGMAS = [0.0, 0.3, 0.6, 1.0, 1.3, 1.5, 2.0, 2.3, 2.6]


def problem(B, H, W, seed):
    prs = [make_problem(H, W, 5, True, 0.01, 0.06, seed + i) for i in range(B)]
    return [to_dev(np.stack([p[k] for p in prs])) for k in ("u_init", "mask", "known")]


@pytest.mark.parametrize("sigma", SIGMAS)
@pytest.mark.parametrize("H,W", [(1, 60), (64, 61), (66, 64), (67, 43), (132, 59), (133, 130), (200, 3),
                                 (65, 250), (71, 180), (300, 64)])
def test_narrow_strips_equal_tiles(H, W, sigma):
    announce(f"narrow strips vs tiles {H}x{W} sigma={sigma}")
    u0, mask, known = problem(2, H, W, 500 + H + W)
    gu = torch.from_numpy(np.random.default_rng(H * W).standard_normal((2, H, W)).astype(np.float32)).cuda()
    out = {}
    for shape in (3, 0):
        p = eed4.params(0.03, sigma, 0.05, 3, 1, flags=eed4.EED4_FORCE_SHAPE(shape))
        u, sums = u0.clone(), torch.zeros((2, 2), dtype=torch.float64, device="cuda")
        eed4.eed4_fsi_cycle(u, mask, known, p, sums)
        # all strips take the same reverse shape here but 3 and 0, which agree bitwise
        g = [torch.empty_like(gu), torch.empty_like(gu), torch.empty(2, device="cuda")]
        eed4.eed4_backward(u0[None].contiguous(), mask, known, p, 1, gu, *g)
        torch.cuda.synchronize()
        out[shape] = u, g[0], g[1], sums.cpu().numpy()
    for i in range(3):
        assert torch.equal(out[3][i], out[0][i]), i
    np.testing.assert_allclose(out[3][3], out[0][3], rtol=1e-12, atol=0)


@pytest.mark.parametrize("sigma", [0.3, 1.0, 2.6])
@pytest.mark.parametrize("sizes", [[(64, 61), (200, 43), (1, 60), (133, 130)], [(67, 64)] * 3])
def test_narrow_strips_in_the_queue(sizes, sigma):
    announce(f"narrow strips, batched {sizes} sigma={sigma}")
    prs = [problem(1, h, w, 600 + i) for i, (h, w) in enumerate(sizes)]
    res = []
    for shape in (3, 5):
        ims = [(u[0].clone(), m[0], k[0], 0.03 + 0.01 * i) for i, (u, m, k) in enumerate(prs)]
        st = eed4.eed4_inpaint_batched(ims, eed4.params(0.03, sigma, 0.05, 4, 3,
                                                        flags=eed4.EED4_FORCE_SHAPE(shape)))
        torch.cuda.synchronize()
        res.append(([im[0] for im in ims], [s.residual for s in st]))
    for a, b in zip(res[0][0], res[1][0]):
        assert torch.equal(a, b)
    np.testing.assert_allclose(res[0][1], res[1][1], rtol=1e-12, atol=0)


def test_narrow_images_do_not_run_half_empty_strips():
    # 500 x 128^2: two strips of 124 columns or three of 60.  Measured 0.83 of the time of the
    # 124-column strips of the same height; alternating samples, the best of each
    announce("500 x 128x128, shape 3 against shape 7")
    u = torch.rand((500, 128, 128), device="cuda")
    mask, out = (u < 0.05).to(torch.uint8), torch.empty_like(u)
    p = {s: eed4.params(0.03, 1.0, 0.05, 15, 1, flags=eed4.EED4_FORCE_SHAPE(s)) for s in (3, 7)}
    best = {3: 1e9, 7: 1e9}
    for _ in range(12):
        for s in (3, 7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            eed4.eed4_fsi_step(u, u, out, mask, p[s], 1)
            a.record()
            for _ in range(20):
                eed4.eed4_fsi_step(u, u, out, mask, p[s], 1)
            b.record()
            b.synchronize()
            best[s] = min(best[s], a.elapsed_time(b) / 20)
    print(f"shape 3 {1e3 * best[3]:.1f} us, shape 7 {1e3 * best[7]:.1f} us")
    assert best[3] < 0.93 * best[7]


@pytest.mark.parametrize("sigma", [0.6, 2.6])
def test_untuned_images_of_32_columns_do_not_run_half_empty_tiles(sigma):
    # 64 x 1200x32 before any tuning: two 32 x 32 tiles across, the second with 4 columns of 28, took
    # 1.35 to 1.4 of the time of 8-row strips
    announce(f"64 x 1200x32 untuned against its strips and tiles, sigma={sigma}")
    u = torch.rand((64, 1200, 32), device="cuda")
    mask = (u < 0.05).to(torch.uint8)
    out = {}
    best = {}
    for _ in range(12):
        for s in (None, 6, 2):
            p = eed4.params(0.03, sigma, 0.05, 15, 1, flags=0 if s is None else eed4.EED4_FORCE_SHAPE(s))
            out[s] = torch.empty_like(u)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            eed4.eed4_fsi_step(u, u, out[s], mask, p, 1)
            a.record()
            for _ in range(20):
                eed4.eed4_fsi_step(u, u, out[s], mask, p, 1)
            b.record()
            b.synchronize()
            best[s] = min(best.get(s, 1e9), a.elapsed_time(b) / 20)
    print(" ".join(f"{s}: {1e3 * t:.1f} us" for s, t in best.items()))
    assert torch.equal(out[None], out[6]) and torch.equal(out[None], out[2])
    assert best[None] < 1.1 * min(best[6], best[2])
