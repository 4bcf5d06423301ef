"""The batched coarse step of the equations with variable velocities against the
oracle, FP64 to 1e-12, at every patch size: two coarse steps of three levels, the
finest inside the domain and (patches up to 32 x 32) across its boundary, where
the rotation's field is not periodic."""
import os

import numpy as np
import pytest

import afsynth
import oracle
import paper_2205_07572_amd as af
from harness import KINDS, closed_masks, rel_linf
from test_gpu_amr_variable import N0, THREE
from test_gpu_amr_wrap import _shift

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.mark.parametrize("where,m", [(w, m) for m in (8, 16, 32, 64, 128) for w in ("inside", "boundary")
                                     if w == "inside" or m <= 32])
@pytest.mark.parametrize("eq", ["rotation", "swirl", "burgers"])
def test_batched_step_matches_oracle(eq, where, m):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    leaves = THREE if where == "inside" else _shift(THREE)
    omega = 1.0 if eq == "rotation" else 0.0
    kw = {"rotation": dict(eq=af.ROTATION, x0=-1.0, y0=-1.0, lx=2.0, ly=2.0, omega=omega),
          "swirl": dict(eq=af.SWIRL), "burgers": dict(eq=af.BURGERS, qmax=1.0)}[eq]
    P = af.Problem(m=m, n0x=N0, n0y=N0, lmax=2, **kw)
    ctx = af.Context(P)
    h = af.Hierarchy(ctx, leaves)
    # smooth periodic data (a jump's image in a foot's cell would decide the error)
    w = 2 * np.pi / P.lx

    def dofs(l, ix, iy):
        i = np.arange(m + 5) - 2.0
        dx = P.dx(l)
        out = {}
        for k in KINDS:
            x = P.x0 + (ix * m + i + (0.5 if k in ("avg", "yedge") else 0.0)) * dx
            y = P.y0 + (iy * m + i + (0.5 if k in ("avg", "xedge") else 0.0)) * dx
            out[k] = (0.4 + 0.2 * np.sin(w * x)[None, :] * np.cos(w * y)[:, None])[None]
        return out

    blocks = [dofs(*l) for l in leaves]
    b0 = af.blocks_to_state(ctx, blocks)
    bufs = [b0, torch.zeros_like(b0)]
    reg = torch.zeros((len(leaves), 4, m, 1), dtype=torch.float64, device="cuda")
    dt0 = 0.4 * P.dx(0) / (1.5 if eq == "rotation" else 1.0)
    mask = ctx.amr_coarse_steps(h, bufs, 0, dt0, 2, reg)
    torch.cuda.synchronize()
    g = [af.state_to_blocks(ctx, b) for b in bufs]
    got = [g[(mask >> l) & 1][k] for k, (l, _, _) in enumerate(leaves)]
    o = oracle.Hier(P.eq, m, N0, N0, 2, x0=P.x0, y0=P.y0, lx=P.lx, ly=P.ly, omega=omega)
    o.set_leaves(leaves)
    for k, b in enumerate(blocks):
        o.set_block(k, b)
    o.fill(0, 0)
    o.run(dt0, 2)
    err = rel_linf(got, [o.get_block(k) for k in range(len(leaves))], closed_masks(m))
    assert err.max() <= TOL, err
