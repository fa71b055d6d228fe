"""Launches of more workgroups than one grid can have (2^32 threads; the runtime runs only the
remainder of a larger one): batches of millions of tiny images, and a work queue of more items than
workgroups.  Tiles, which need a workgroup to an image, must equal the strips, which need a quarter
of that and stay below the limit."""
import numpy as np
import pytest

from tests.helpers import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
import paper_2006_10406_amd as eed4  # noqa: E402

B = 2 ** 24 + 5                         # one 256-thread workgroup each: 2^32 + 1280 threads


@pytest.fixture(scope="module")
def images():
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda: torch.rand((B, 1, 2), generator=g, device="cuda")
    u, prev = rnd(), rnd()
    mask = (torch.rand((B, 1, 2), generator=g, device="cuda") < 0.25).to(torch.uint8)
    return u, prev, mask


@pytest.mark.parametrize("shape", [0, 2, 10])
def test_steps_and_cycles_cover_millions_of_images(images, shape):
    announce(f"{B} images of 1x2, shape {shape}")
    u, prev, mask = images
    out = {}
    for s in (shape, 5):
        p = eed4.params(0.03, 0.5, 0.05, 2, 1, flags=eed4.EED4_FORCE_SHAPE(s))
        o, v = torch.full_like(u, -7.0), u.clone()
        eed4.eed4_fsi_step(u, prev, o, mask, p, 1)
        sums = torch.full((B, 2), -7.0, dtype=torch.float64, device="cuda")
        eed4.eed4_fsi_cycle(v, mask, u, p, sums)
        torch.cuda.synchronize()
        out[s] = o, v, sums
    assert torch.equal(out[shape][0], out[5][0]) and torch.equal(out[shape][1], out[5][1])
    du = out[5][1].double() - u.double()
    want = torch.stack([(du * du).sum((1, 2)), (out[5][1].double() ** 2).sum((1, 2))], 1)
    for s in (shape, 5):                # two FP64 terms to a sum
        assert torch.allclose(out[s][2], want, rtol=1e-14, atol=0)


@pytest.mark.parametrize("shape", [1, 2])
def test_backward_covers_millions_of_images(images, shape):
    announce(f"backward of {B} images of 1x2, shape {shape}")
    u, prev, mask = images
    out = {}
    for s in (shape, 5):
        p = eed4.params(0.03, 0.5, 0.05, 2, 1, flags=eed4.EED4_FORCE_SHAPE(s))
        g = [torch.full_like(u, -7.0), torch.full_like(u, -7.0), torch.full((B,), -7.0, device="cuda")]
        eed4.eed4_backward(u[None], mask, u, p, 1, prev, *g)
        torch.cuda.synchronize()
        out[s] = g
    for i in (0, 1):
        assert torch.equal(out[shape][i], out[5][i])
    # images of one row have no gradient across it: dL/dlambda comes from two pixels of a row
    assert torch.allclose(out[shape][2], out[5][2], rtol=1e-4, atol=1e-7)
    assert not (out[shape][2] == -7.0).any()


def test_batched_queue_beyond_one_grid():
    # 2 x 40000 x 41900 pixels are 17.5 million 16 x 16 tiles
    free, _ = torch.cuda.mem_get_info()
    if free < 90 * 2 ** 30:
        pytest.skip(f"needs about 90 GiB of free device memory, {free / 2 ** 30:.0f} GiB free")
    H, W = 40000, 41900
    announce(f"batched 2 x {H}x{W} on 16 x 16 tiles")
    ims = []
    for i in range(2):
        u = torch.empty((H, W), device="cuda")
        for r in range(0, H, 4000):     # in parts: torch's generator indexes 32 bits
            u[r:r + 4000].uniform_(0.0, 1.0)
        mask = torch.empty((H, W), dtype=torch.uint8, device="cuda")
        for r in range(0, H, 4000):
            mask[r:r + 4000].copy_(u[r:r + 4000] < 0.05)
        ims.append((u, mask))
    known = [u.clone() for u, _ in ims]
    res = {}
    for s in (10, 5):
        p = eed4.params(0.03, 0.5, 0.05, 2, 1, flags=eed4.EED4_FORCE_SHAPE(s))
        us = [k.clone() for k in known]
        eed4.eed4_inpaint_batched([(us[i], ims[i][1], known[i], 0.03) for i in range(2)], p)
        torch.cuda.synchronize()
        res[s] = us
    for i in range(2):
        for r in range(0, H, 4000):
            assert torch.equal(res[10][i][r:r + 4000], res[5][i][r:r + 4000]), (i, r)
    del res, known, ims
    torch.cuda.empty_cache()
