"""Graph replay after an option of the context has changed: the replay must be
of the schedule that the option asks for, seen in the buffer that holds level F
in the middle of a coarse step (written without fused pairs only)."""
import os

import numpy as np
import pytest

import afsynth
import paper_2205_07572_amd as af
from harness import KINDS
from test_gpu_amr_variable import N0, THREE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eq", ["acoustics", "advection", "swirl"])
def test_fused_pairs_toggle(eq):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    m = 8
    kw = {"acoustics": dict(eq=af.ACOUSTICS, c=1.0), "advection": dict(eq=af.ADVECTION, a=1.0, b=0.5),
          "swirl": dict(eq=af.SWIRL)}[eq]
    P = af.Problem(prec=af.FP64, m=m, n0x=N0, n0y=N0, lmax=2, **kw)
    ctx = af.Context(P)
    h = af.Hierarchy(ctx, THREE)
    rng = np.random.default_rng(1)
    init = af.blocks_to_state(ctx, [{k: rng.uniform(0.2, 0.6, (P.ncomp, m + 5, m + 5)) for k in KINDS} for _ in THREE])
    bufs = [init.clone(), torch.zeros_like(init)]
    reg = torch.zeros((len(THREE), 4, m, P.ncomp), dtype=torch.float64, device="cuda")

    def step(graph):
        bufs[0].copy_(init)
        bufs[1].zero_()
        ctx.amr_coarse_step(h, bufs, 0, 0.4 * P.dx(0), reg, use_graph=graph, t0=0.2)
        torch.cuda.synchronize()
        return [b.clone() for b in bufs]

    seen = []
    for fused in (True, False, True):
        ctx.fused_pairs = fused
        eager, replay = step(False), step(True)
        assert all(torch.equal(a, b) for a, b in zip(eager, replay)), fused
        seen.append(eager)
    # the two schedules can be told apart
    assert not all(torch.equal(a, b) for a, b in zip(seen[0], seen[1]))
