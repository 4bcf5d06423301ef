"""How many launches the level advance takes: as few as its shapes allow (the bit
of the level in the mask flips with each), for step counts that are no multiple
of anything."""
import os

import pytest

import afsynth
import paper_2205_07572_amd as af

pytestmark = pytest.mark.gpu


def fewest(ks, n):
    """The fewest numbers of ks (with repetition) that add up to n."""
    best = [0] + [n + 1] * n
    for r in range(1, n + 1):
        best[r] = 1 + min(best[r - k] for k in ks if k <= r)
    return best[n]


@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("m,n", [(16, 3), (16, 16), (32, 3), (32, 16)])
def test_fewest_launches(m, n, prec):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    P = af.Problem(eq=af.ADVECTION, prec=prec, m=m, n0x=n, n0y=n, a=1.0, b=0.5)
    ctx = af.Context(P)
    h = af.Hierarchy(ctx, afsynth.uniform_leaves(n, n, 0))
    bufs = [ctx.new_state(n * n), ctx.new_state(n * n)]
    # up to 256 patches: every length up to the longest
    ks = {k for k, _ in ctx.advance_shapes()}
    if prec == af.FP64 and m == 32:
        assert max(ks) == 12
    for steps in range(1, 3 * max(ks) + 1):
        mask = ctx.level_advance(h, bufs, 0, 0, 0.4 * P.dx(0), steps)
        assert mask == fewest(ks, steps) % 2, steps
    for steps in (100, 257):  # full lengths and the rest of the last three
        bufs[0].uniform_(-1.0, 1.0)
        bufs[1].zero_()
        mask = ctx.level_advance(h, bufs, 0, 0, 0.4 * P.dx(0), steps)
        torch.cuda.synchronize()
        assert float(bufs[mask & 1][0, :, :, 2:2 + m, 2:2 + m].abs().max()) > 0
