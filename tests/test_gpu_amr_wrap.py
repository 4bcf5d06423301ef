"""Fused pairs of the batched coarse step where the finest level lies inside
the domain and where it straddles the periodic boundary, for the equations
with variable velocities: bit for bit the step without fused pairs, which in
turn follows the recursion of Sec. 3.2.  The rotation's field is not periodic,
nor is the swirl's on a domain that is no whole number of periods long, so
across the boundary a patch and its neighbour evaluate a shared position from
different coordinates."""
import os

import numpy as np
import pytest

import afsynth
import paper_2205_07572_amd as af
from harness import KINDS, closed_masks
from test_gpu_amr_variable import N0, THREE, _recursion

pytestmark = pytest.mark.gpu


def _shift(leaves):
    """The leaf set moved by half the domain in both directions."""
    return afsynth.sort_leaves([(l, (i + (N0 << l) // 2) % (N0 << l), (j + (N0 << l) // 2) % (N0 << l))
                                for l, i, j in leaves])


# the shifted domains have cell boundaries that are no short binary fractions
EQS = {"rotation": dict(eq=af.ROTATION, x0=-1.0, y0=-1.0, lx=2.0, ly=2.0, omega=1.0),
       "rotation_shifted": dict(eq=af.ROTATION, x0=-0.9, y0=-1.1, lx=1.9, ly=1.9, omega=1.0),
       "swirl": dict(eq=af.SWIRL), "swirl_shifted": dict(eq=af.SWIRL, x0=0.1, y0=0.3),
       "swirl_1.5": dict(eq=af.SWIRL, x0=0.1, lx=1.5, ly=1.5),
       "burgers": dict(eq=af.BURGERS, qmax=1.0)}


@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("m", [8, 16])
@pytest.mark.parametrize("where", ["inside", "boundary"])
@pytest.mark.parametrize("eq", list(EQS))
def test_fused_pairs(eq, where, m, prec):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    leaves = THREE if where == "inside" else _shift(THREE)
    P = af.Problem(prec=prec, m=m, n0x=N0, n0y=N0, lmax=2, **EQS[eq])
    rng = np.random.default_rng(m)
    blocks = [{k: rng.uniform(0.2, 0.6, (1, m + 5, m + 5)) for k in KINDS} for _ in leaves]
    t0, dt0 = 0.2, 0.4 * P.dx(0) / (1.5 if P.eq == af.ROTATION else 1.0)
    closed = closed_masks(m)
    out = {}
    for name in ("recursion", "unfused", "fused"):
        ctx = af.Context(P)
        ctx.fused_pairs = name == "fused"
        h = af.Hierarchy(ctx, leaves)
        b0 = af.blocks_to_state(ctx, blocks)
        bufs = [b0, torch.zeros_like(b0)]
        ctx.ghost_fill(h, bufs, 0, 0, 0)
        reg = torch.zeros((len(leaves), 4, m, 1), dtype=torch.float64, device="cuda")
        if name == "recursion":
            mask = _recursion(ctx, h, bufs, reg, t0, dt0)
        else:
            mask = ctx.amr_coarse_steps(h, bufs, 0, dt0, 2, reg, t0=t0)
        torch.cuda.synchronize()
        g = [af.state_to_blocks(ctx, b) for b in bufs]
        out[name] = [g[(mask >> l) & 1][k] for k, (l, _, _) in enumerate(leaves)]

    def diff(a, b):
        return max(np.abs(out[a][i][k][0][closed[k]] - out[b][i][k][0][closed[k]]).max()
                   for i in range(len(leaves)) for k in KINDS)

    # a foot is known to a few roundings of its position (FP64) or of its
    # displacement (FP32), a value moves by about 4 per cell, in 8 substeps
    # that amplify 3 times at most
    eps = 2.0 ** -53 * 16 * m * N0 if prec == af.FP64 else 2.0 ** -24 * 4 * 4
    for name in ("unfused", "fused"):
        assert diff(name, "recursion") <= 4 * 8 * 3 * eps, name
    assert diff("fused", "unfused") == 0.0
