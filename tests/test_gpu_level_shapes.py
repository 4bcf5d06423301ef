"""The shape that the level advance chooses by itself, on both sides of the
patch counts at which the choice changes (256, 768, 1536, 8192), for launches of
full length and tails, against the one-step shape set on the context."""
import os

import pytest

import afsynth
import paper_2205_07572_amd as af

pytestmark = pytest.mark.gpu

CASES = [("advection", m, n, v) for m in (16, 32) for n in ((3, 5), (16, 16), (16, 17), (24, 32), (25, 32), (25, 64))
         for v in ((0.8, 0.5), (-0.8, 0.5))]
CASES += [("acoustics", 16, n, None) for n in ((3, 5), (16, 16), (16, 17), (64, 128), (65, 128))]
CASES += [("acoustics", 32, n, None) for n in ((3, 5), (16, 17))]


@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("eq,m,n,v", CASES)
def test_chosen_shape(eq, m, n, v, prec):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    if eq == "acoustics" and m == 32 and prec == af.FP64:
        pytest.skip("no shape is compiled for it")
    kw = dict(eq=af.ADVECTION, a=v[0], b=v[1]) if eq == "advection" else dict(eq=af.ACOUSTICS, c=1.0)
    P = af.Problem(prec=prec, m=m, n0x=n[0], n0y=n[1], lmax=0, lx=float(n[0]), ly=float(n[1]), **kw)
    torch.manual_seed(1)
    start, ref = None, None
    # the first context takes one step per launch
    for one_step in (True, False):
        ctx = af.Context(P)
        if one_step:
            ctx.set_advance_shape(*min(ctx.advance_shapes()))
        h = af.Hierarchy(ctx, afsynth.uniform_leaves(n[0], n[1], 0))
        if start is None:
            start = ctx.new_state(n[0] * n[1])
            start.uniform_(-1.0, 1.0)
        got = []
        for nsteps in ((1, 7, 30) if eq == "advection" else (1, 5)):
            bufs = [start.clone(), torch.zeros_like(start)]
            mask = ctx.level_advance(h, bufs, 0, 0, 0.4 * P.dx(0), nsteps)
            torch.cuda.synchronize()
            s = bufs[mask & 1][..., 2:2 + m, 2:2 + m]  # interior cells, low nodes
            got.append((nsteps, s.double()))
        if one_step:
            ref = got
            continue
        # rounding of about 10 operations of weight 1 per step, in random order
        eps = 2.0 ** -53 if prec == af.FP64 else 2.0 ** -24
        for (nsteps, a), (_, b) in zip(ref, got):
            err = float((a - b).abs().max()) / float(a.abs().max())
            assert err <= 16 * eps * nsteps, (nsteps, err)
