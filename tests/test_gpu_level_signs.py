"""The level advance over the signs of the velocity and at the edges of the
upwind source pattern (a zero component, a directional Courant number of 1/2),
on a rectangular patch grid, against the oracle's periodic grid: interior
averages and every node of the closed squares, hi lines included."""
import os

import numpy as np
import pytest

import afsynth
import oracle
import paper_2205_07572_amd as af
from tests.harness import KINDS

pytestmark = pytest.mark.gpu

# (a, b, Courant number of the faster direction): mirrored in x, in y, in
# both; the pattern's edge from below and at it; a component of zero
VELOCITY = [(-1.0, 0.5, 0.4), (0.6, -0.9, 0.45), (-0.7, -0.8, 0.4), (-1.0, 1.0, 0.4999), (-1.0, 0.9, 0.5),
            (-1.0, 0.0, 0.4), (0.0, -1.0, 0.3)]


@pytest.mark.parametrize("m", [16, 32])
@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("a,b,cfl", VELOCITY)
def test_velocity_signs(a, b, cfl, prec, m):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    nx, ny = 3, 5
    prob = af.Problem(eq=af.ADVECTION, prec=prec, m=m, n0x=nx, n0y=ny, a=a, b=b)
    ctx = af.Context(prob)
    h = af.Hierarchy(ctx, afsynth.uniform_leaves(nx, ny, 0))
    d0 = afsynth.dofs_periodic(afsynth.fourier_modes(4), nx * m, ny * m, nq=4)
    if prec == af.FP32:
        d0 = {k: (v.astype(np.float32).astype(np.float64) if isinstance(v, np.ndarray) else v) for k, v in d0.items()}
    blk = afsynth.periodic_to_blocks(d0, m)
    b0 = af.blocks_to_state(ctx, [{k: blk[k][p] for k in KINDS} for p in range(nx * ny)])
    bufs = [b0, torch.zeros_like(b0)]
    dt = cfl / max(abs(a) / prob.dx(0), abs(b) / prob.dy(0))
    nsteps = 11  # a whole launch and tails
    mask = ctx.level_advance(h, bufs, 0, 0, dt, nsteps)
    torch.cuda.synchronize()
    got = bufs[mask & 1].double().cpu().numpy()[:, 0]
    ref = oracle.run_periodic(0, d0, dt, nsteps, a=a, b=b)
    scale = max(np.abs(ref[k]).max() for k in KINDS)
    # FP64: 1e-12; FP32: about 5 units of rounding (6e-8) per step
    tol = 1e-12 if prec == af.FP64 else 3e-7 * nsteps
    for q, k in enumerate(KINDS):
        rows, cols = m + (k in ("corner", "yedge")), m + (k in ("corner", "xedge"))
        for p in range(nx * ny):
            gj = (p // nx * m + np.arange(rows)) % (ny * m)
            gi = (p % nx * m + np.arange(cols)) % (nx * m)
            err = np.abs(got[q, p, 2:2 + rows, 2:2 + cols] - ref[k][0][gj[:, None], gi[None, :]]).max() / scale
            assert err <= tol, (k, p, err)
