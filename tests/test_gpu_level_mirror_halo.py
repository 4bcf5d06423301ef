"""The long shapes of the mirrored one-pass level advance against the oracle's
periodic grid, interior averages and the closed squares with their high lines.
Each patch's high lines and ghost layers are NaN at the start: a step reads a
DOF from the patch that owns it, also where the halo is as wide as a patch
(K = m) and the owner two patches on, on grids one and two patches wide too."""
import os

import numpy as np
import pytest

import afsynth
import oracle
import paper_2205_07572_amd as af
from harness import KINDS

pytestmark = pytest.mark.gpu

GRIDS = [(3, 5), (1, 4), (2, 1)]


@pytest.mark.parametrize("a,b", [(-1.0, 0.5), (0.6, -0.9), (-0.7, -0.8)])
@pytest.mark.parametrize("prec,m", [(af.FP32, 16), (af.FP64, 16), (af.FP32, 32), (af.FP64, 32)],
                         ids=["fp32-16", "fp64-16", "fp32-32", "fp64-32"])
def test_mirrored_long_shapes(prec, m, a, b):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    for nx, ny in GRIDS:
        prob = af.Problem(eq=af.ADVECTION, prec=prec, m=m, n0x=nx, n0y=ny, lx=float(nx), ly=float(ny), a=a, b=b)
        d0 = afsynth.dofs_periodic(afsynth.fourier_modes(4), nx * m, ny * m, nq=4)
        d0["dx"], d0["dy"] = prob.dx(0), prob.dy(0)
        if prec == af.FP32:
            d0 = {k: (v.astype(np.float32).astype(np.float64) if isinstance(v, np.ndarray) else v)
                  for k, v in d0.items()}
        blk = afsynth.periodic_to_blocks(d0, m)
        ctx = af.Context(prob)
        init = af.blocks_to_state(ctx, [{k: blk[k][p] for k in KINDS} for p in range(nx * ny)])
        own = init[..., 2:2 + m, 2:2 + m].clone()
        init.fill_(float("nan"))
        init[..., 2:2 + m, 2:2 + m] = own
        dt = 0.45 / max(abs(a) / prob.dx(0), abs(b) / prob.dy(0))
        refs = {}
        for K, nt in ctx.advance_shapes_upwind():
            ctx = af.Context(prob)
            ctx.set_advance_shape(K, nt)
            h = af.Hierarchy(ctx, afsynth.uniform_leaves(nx, ny, 0))
            bufs = [init.clone(), torch.full_like(init, float("nan"))]
            mask = ctx.level_advance(h, bufs, 0, 0, dt, K)
            torch.cuda.synchronize()
            assert mask == 1
            got = bufs[mask & 1].double().cpu().numpy()[:, 0]
            if K not in refs:
                refs[K] = oracle.run_periodic(0, d0, dt, K, a=a, b=b)
            ref = refs[K]
            scale = max(np.abs(ref[k]).max() for k in KINDS)
            # FP64: 1e-12; FP32: about 5 units of rounding (6e-8) per step
            tol = 1e-12 if prec == af.FP64 else 3e-7 * K
            for q, k in enumerate(KINDS):
                rows, cols = m + (k in ("corner", "yedge")), m + (k in ("corner", "xedge"))
                for p in range(nx * ny):
                    gj = (p // nx * m + np.arange(rows)) % (ny * m)
                    gi = (p % nx * m + np.arange(cols)) % (nx * m)
                    d = np.abs(got[q, p, 2:2 + rows, 2:2 + cols] - ref[k][0][gj[:, None], gi[None, :]])
                    err = d.max() / scale  # NaN if a value is
                    assert err <= tol, ((nx, ny), (K, nt), k, p, err)
