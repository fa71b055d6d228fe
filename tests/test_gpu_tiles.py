"""Workgroup-tile step kernels at the edges of their tiles: one cycle, residual included, must
equal the strip kernel's bitwise (all shapes form every value the same way); the tensor variants'
tiles likewise against their strips.  The strips are compared with the FP64 oracle elsewhere."""
import numpy as np
import pytest

from synth import make_problem
from tests.helpers import announce, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
import paper_2006_10406_amd as eed4  # noqa: E402


def cycle(b, sigma, n, flags):
    u = to_dev(b["u_init"])
    sums = torch.zeros((u.shape[0], 2), dtype=torch.float64, device="cuda")
    eed4.eed4_fsi_cycle(u, to_dev(b["mask"]), to_dev(b["known"]),
                        eed4.params(0.03, sigma, 0.05, n, 1, flags=flags), sums)
    torch.cuda.synchronize()
    return u.cpu().numpy(), sums.cpu().numpy()


def batch(B, H, W, seed):
    prs = [make_problem(H, W, 5, True, 0.01, 0.06, seed + i) for i in range(B)]
    return {k: np.stack([p[k] for p in prs]) for k in ("u_init", "mask", "known")}


@pytest.mark.parametrize("sigma", [0.0, 0.3, 0.6, 1.0, 1.3, 1.5, 2.0, 2.3, 2.6])
@pytest.mark.parametrize("H,W", [(32, 60), (33, 61), (31, 59), (16, 28), (17, 29), (65, 121),
                                 (1, 64), (64, 1), (4, 90), (90, 5), (40, 75), (100, 240)])
def test_tile_shapes_equal_strips(H, W, sigma):
    announce(f"tiles vs strips {H}x{W} sigma={sigma}")
    b = batch(2, H, W, 40 + H + W)
    ref = cycle(b, sigma, 3, eed4.EED4_FORCE_SHAPE(5))
    for shape in eed4.TILE_SHAPES:
        got = cycle(b, sigma, 3, eed4.EED4_FORCE_SHAPE(shape))
        assert np.array_equal(got[0], ref[0]), eed4.SHAPE_NAMES[shape]
        # the FP64 residual partials group the pixels differently: equal to FP64 rounding of a
        # sum of H*W terms
        np.testing.assert_allclose(got[1], ref[1], rtol=1e-12, atol=0)


@pytest.mark.parametrize("d,r", [(0, 1), (1, 0), (2, 1), (3, 2)])
@pytest.mark.parametrize("B,H,W,sigma", [(1, 33, 61, 2.0), (2, 75, 130, 1.0), (16, 515, 301, 1.5)])
def test_variant_tiles_equal_variant_strips(B, H, W, sigma, d, r):
    # the sizes take the 16-row tiles (twice) and the 32-row tiles of the variants' size rule
    fl = eed4.EED4_DIFFUSIVITY(d) | eed4.EED4_MU3(r)
    announce(f"variant {d}/{r} tiles vs strips {B} x {H}x{W} sigma={sigma}")
    b = batch(B, H, W, 70 + H)
    ref = cycle(b, sigma, 2, fl | eed4.EED4_FORCE_SHAPE(5))
    got = cycle(b, sigma, 2, fl)
    assert np.array_equal(got[0], ref[0])
    np.testing.assert_allclose(got[1], ref[1], rtol=1e-12, atol=0)


@pytest.mark.parametrize("sigma", [0.0, 0.3, 1.0, 1.5, 2.0, 2.6])
@pytest.mark.parametrize("H,W", [(10, 48), (34, 49), (35, 97), (24, 54), (25, 55), (1, 70), (70, 1),
                                 (3, 3), (120, 130)])
def test_reverse_tiles_equal_reverse_strips(H, W, sigma):
    # all reverse shapes form every value the same way: gradients of f and u_init bitwise equal
    # (dL/dlambda sums the same terms in another grouping; the oracle tests bound it)
    announce(f"reverse tiles vs strips {H}x{W} sigma={sigma}")
    b = batch(2, H, W, 90 + H + W)
    mask, known = to_dev(b["mask"]), to_dev(b["known"])
    gu = torch.from_numpy(np.random.default_rng(H * W).standard_normal((2, H, W)).astype(np.float32)).cuda()
    out = {}
    for shape in (6, 0, 1, 2):
        p = eed4.params(0.03, sigma, 0.05, 3, 2, flags=eed4.EED4_FORCE_SHAPE(shape))
        u = to_dev(b["u_init"])
        ck = torch.empty((2, 2, H, W), device="cuda")
        eed4.eed4_inpaint(u, mask, known, p, ckpt=ck)
        g = [torch.empty_like(gu), torch.empty_like(gu), torch.empty(2, device="cuda")]
        eed4.eed4_backward(ck, mask, known, p, 2, gu, *g)
        torch.cuda.synchronize()
        out[shape] = g
    for shape in (0, 1, 2):
        assert torch.equal(out[shape][0], out[6][0]) and torch.equal(out[shape][1], out[6][1]), shape
        assert torch.isfinite(out[shape][2]).all()


@pytest.mark.parametrize("sigma", [0.0, 0.3, 0.6, 1.0, 1.3, 1.5, 2.0, 2.3, 2.6])
@pytest.mark.parametrize("H,W", [(28, 124), (29, 125), (57, 126), (65, 127), (60, 249), (3, 251),
                                 (137, 123), (140, 1), (1, 400), (200, 380)])
def test_tall_strips_equal_tiles(H, W, sigma):
    # 124-column strips at their column and segment edges: strips inside the image (8-byte
    # accesses, odd widths included), strips at and over its borders, segments in both directions
    announce(f"tall strips vs tiles {H}x{W} sigma={sigma}")
    b = batch(2, H, W, 20 + H + W)
    mask, known = to_dev(b["mask"]), to_dev(b["known"])
    ref = cycle(b, sigma, 3, eed4.EED4_FORCE_SHAPE(0))
    gu = torch.from_numpy(np.random.default_rng(H * W).standard_normal((2, H, W)).astype(np.float32)).cuda()
    grads = {}
    for shape in (0, 3, 4, 7, 8):
        fl = eed4.EED4_FORCE_SHAPE(shape)
        got = cycle(b, sigma, 3, fl)
        assert np.array_equal(got[0], ref[0]), eed4.SHAPE_NAMES[shape]
        np.testing.assert_allclose(got[1], ref[1], rtol=1e-12, atol=0)
        # the backward's recompute runs them too, keeping K_sigma * u^k
        p = eed4.params(0.03, sigma, 0.05, 3, 1, flags=fl)
        ck = to_dev(b["u_init"])[None].contiguous()
        g = [torch.empty_like(gu), torch.empty_like(gu), torch.empty(2, device="cuda")]
        eed4.eed4_backward(ck, mask, known, p, 1, gu, *g)
        torch.cuda.synchronize()
        grads[shape] = g
    for shape in (3, 4, 7, 8):
        for i in (0, 1):
            assert torch.equal(grads[shape][i], grads[0][i]), eed4.SHAPE_NAMES[shape]
