"""The acoustic level advance (one step, or a fused pair, per launch in the
orbit form) on rectangular patch grids, odd step counts and unequal cell
sides, against the oracle's periodic grid over the closed squares, hi lines
included; and captured as the first call of its context, replayed three times
with eager work between."""
import os

import numpy as np
import pytest

import afsynth
import oracle
import paper_2205_07572_amd as af
from tests.harness import KINDS

pytestmark = pytest.mark.gpu


def _setup(m, prec, nx, ny, ly):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    prob = af.Problem(eq=af.ACOUSTICS, prec=prec, m=m, n0x=nx, n0y=ny, ly=ly, c=1.3)
    ctx = af.Context(prob)
    h = af.Hierarchy(ctx, afsynth.uniform_leaves(nx, ny, 0))
    rng = np.random.default_rng(m + nx)
    d0 = {k: rng.standard_normal((3, ny * m, nx * m)) for k in KINDS}
    if prec == af.FP32:
        d0 = {k: v.astype(np.float32).astype(np.float64) for k, v in d0.items()}
    d0["dx"], d0["dy"] = prob.dx(0), prob.dy(0)
    blk = afsynth.periodic_to_blocks(d0, m)
    b0 = af.blocks_to_state(ctx, [{k: blk[k][p] for k in KINDS} for p in range(nx * ny)])
    return torch, prob, ctx, h, d0, [b0, torch.zeros_like(b0)]


@pytest.mark.parametrize("m,prec,nx,ny,ly,nsteps", [
    (16, af.FP64, 1, 1, 1.0, 3), (16, af.FP64, 3, 2, 0.5, 5), (16, af.FP32, 2, 5, 2.0, 4), (16, af.FP32, 3, 3, 1.0, 1),
    (32, af.FP32, 2, 3, 1.0, 3)])
def test_closed_squares(m, prec, nx, ny, ly, nsteps):
    torch, prob, ctx, h, d0, bufs = _setup(m, prec, nx, ny, ly)
    dt = 0.45 * min(prob.dx(0), prob.dy(0)) / prob.c
    mask = ctx.level_advance(h, bufs, 0, 0, dt, nsteps)
    torch.cuda.synchronize()
    got = bufs[mask & 1].double().cpu().numpy()
    ref = oracle.run_periodic(1, d0, dt, nsteps, c=prob.c)
    scale = max(np.abs(ref[k]).max() for k in KINDS)
    # FP64 1e-12; FP32 on random data: rounding of sums of 25 terms, about 10 units (6e-8) per step
    tol = 1e-12 if prec == af.FP64 else 6e-7 * nsteps
    for q, k in enumerate(KINDS):
        rows, cols = m + (k in ("corner", "yedge")), m + (k in ("corner", "xedge"))
        for p in range(nx * ny):
            gj = (p // nx * m + np.arange(rows)) % (ny * m)
            gi = (p % nx * m + np.arange(cols)) % (nx * m)
            err = np.abs(got[q, :, p, 2:2 + rows, 2:2 + cols] - ref[k][:, gj[:, None], gi[None, :]]).max() / scale
            assert err <= tol, (k, p, err)


@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
def test_captured_first_call(prec):
    torch, prob, ctx, h, d0, bufs = _setup(16, prec, 3, 2, 1.0)
    dt = 0.4 * min(prob.dx(0), prob.dy(0)) / prob.c
    init = bufs[0].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mask = ctx.level_advance(h, bufs, 0, 0, dt, 5)
    other = af.Context(prob)
    eager = [init.clone(), torch.zeros_like(init)]
    assert other.level_advance(af.Hierarchy(other, afsynth.uniform_leaves(3, 2, 0)), eager, 0, 0, dt, 5) == mask
    torch.cuda.synchronize()
    for _ in range(3):
        bufs[0].copy_(init)
        bufs[1].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(bufs, eager):
            assert torch.equal(a, b)
