"""Traced feet of the variable-velocity equations at the edges of their rules,
one patch step against the oracle's: displacements of up to a whole cell in
every direction (Courant number 1), zero time steps (feet on the nodes), swirl
cells on both sides of the small-angle bound (pi dt = 0.4)."""
import math
import os

import numpy as np
import pytest

import oracle
import paper_2205_07572_amd as af
from harness import KINDS, closed_masks

pytestmark = pytest.mark.gpu
M = 8

CASES = [("rotation", w, c) for w in (math.pi, -2.0) for c in (1.0, 0.3, 0.0)]
CASES += [("burgers", s, c) for s in (1.0, -1.0) for c in (1.0, 0.5, 0.0)]
CASES += [("swirl", l, c) for l in (1.0, 4.0, 0.25) for c in (1.0, 0.6)]


@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("eq,par,cfl", CASES)
def test_feet(eq, par, cfl, prec):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    rng = np.random.default_rng(5)
    kw = {"eq": {"rotation": af.ROTATION, "burgers": af.BURGERS, "swirl": af.SWIRL}[eq], "prec": prec, "m": M,
          "n0x": 2, "n0y": 2}
    if eq == "rotation":
        kw.update(x0=-1.0, y0=-0.5, lx=2.0, ly=2.0, omega=par, xc=0.1, yc=0.2)
    elif eq == "burgers":
        kw.update(qmax=1.0)
    else:
        kw.update(lx=par, ly=par)
    P = af.Problem(**kw)
    dx = P.dx(0)
    # rotation by angle w: |x - xc| <= 0.9 and |y - yc| <= 1.3 in this patch, so a foot is at most
    # 1.3 sin w + 0.9 (1 - cos w) < 1.3 * 1.05 w away along an axis
    speed = 1.0 if eq != "rotation" else abs(par) * 1.3 * 1.05
    dt, t = cfl * dx / speed, 0.15
    blk = {k: rng.uniform(-1, 1, (1, M + 5, M + 5)) for k in KINDS}
    if eq == "burgers":  # constant at Courant number 1 (feet on the next node), else noise around 0 or the speed
        blk = {k: np.full_like(v, par) if cfl == 1.0 else 0.25 * v + 0.5 * par for k, v in blk.items()}
    if prec == af.FP32:
        blk = {k: v.astype(np.float32).astype(np.float64) for k, v in blk.items()}
    ctx = af.Context(P)
    ix, iy = 1, 1
    a = af.blocks_to_state(ctx, [blk])
    b = torch.zeros_like(a)
    xy = torch.tensor([[ix, iy]], dtype=torch.int32, device="cuda")
    ctx.patch_step(a, b, 0, 1, 0, dt, leaf_xy=xy, t=t)
    torch.cuda.synchronize()
    got = af.state_to_blocks(ctx, b)[0]
    x0p, y0p = P.x0 + ix * M * dx, P.y0 + iy * M * dx
    if eq == "rotation":
        ref = oracle.patch_step_rot(M, blk, x0p, y0p, dx, dx, dt, par, P.xc, P.yc)
    elif eq == "swirl":
        ref = oracle.patch_step_swirl(M, blk, x0p, y0p, dx, dx, dt, t)
    else:
        ref = oracle.patch_step_burgers(M, blk, dx, dx, dt)
    ref = ref[0] if isinstance(ref, tuple) else ref
    # FP64 1e-12.  FP32: data of size 1 whose reconstructions bend by O(1) per
    # cell: the foot's coordinate is known to a few roundings (2^-24) of the
    # displacement (rotation, swirl: of positions of size 4 over dx), each
    # moving the value by at most its slope, about 10 per cell; Burgers takes
    # two such evaluations, the first's error times the slope and tau / dx
    pos = 4.0 / dx if eq != "burgers" else 10.0
    tol = 1e-12 if prec == af.FP64 else 40 * 2.0 ** -24 * max(1.0, pos)
    for k in KINDS:
        mk = closed_masks(M)[k]
        err = np.abs(got[k][0][mk] - ref[k][0][mk]).max()
        assert err <= tol * max(1.0, np.abs(ref[k][0][mk]).max()), (k, err)
