"""Checkpoints of a run of a fixed number of cycles: ckpt[m] is bitwise the state after m cycles, and
u and the residual those of the run without checkpoints, on both sides of the size from which cycles
write straight into the next checkpoint (2^19 pixels, 4 cycles)."""
import numpy as np
import pytest

from synth import make_problem
from tests.helpers import announce, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
import paper_2006_10406_amd as eed4  # noqa: E402


@pytest.mark.parametrize("B,H,W", [(2, 511, 513), (1, 725, 723), (2, 512, 513)])
@pytest.mark.parametrize("n,M,history", [(1, 4, False), (2, 4, True), (3, 5, False), (3, 3, False)])
def test_checkpoints_hold_the_start_of_every_cycle(B, H, W, n, M, history):
    announce(f"checkpoints {B} x {H}x{W}, {M} cycles of {n}, history {history}")
    prs = [make_problem(H, W, 5, True, 0.01, 0.06, 300 + i) for i in range(B)]
    u0, mask, known = (to_dev(np.stack([p[k] for p in prs])) for k in ("u_init", "mask", "known"))

    def run(cycles, ckpt=None):
        u = u0.clone()
        st, hist = eed4.eed4_inpaint(u, mask, known, eed4.params(0.03, 1.0, 0.05, n, cycles), ckpt=ckpt,
                                     history=history)
        torch.cuda.synchronize()
        return u, st, hist

    ckpt = torch.full((M, B, H, W), float("nan"), device="cuda")
    u, st, hist = run(M, ckpt)
    ref, rst, rhist = run(M)
    assert torch.equal(u, ref) and st.residual == rst.residual and st.cycles == rst.cycles == M
    if history:
        assert np.array_equal(hist, rhist)
    held = torch.where(mask != 0, known, u0)
    for m in range(M):
        assert torch.equal(ckpt[m], run(m)[0] if m else held), m
