"""The batched coarse step of the equations with variable velocities against
the recursion of Sec. 3.2 made of the library's own patch steps, ghost fills
and conservative fixes: every patch size, both tile heights where there are
two, fused pairs on and off, two levels and three, eager, replayed and two
steps in one call."""
import math
import os

import numpy as np
import pytest

import afsynth
import paper_2205_07572_amd as af
from harness import KINDS, closed_masks

pytestmark = pytest.mark.gpu
N0 = 4
TWO = afsynth.sort_leaves([(0, i, j) for i in range(N0) for j in range(N0) if not (1 <= i <= 2 and j == 1)] +
                          [(1, i, j) for i in range(2, 6) for j in range(2, 4)])
THREE = afsynth.sort_leaves(
    [(0, i, j) for i in range(N0) for j in range(N0) if not (1 <= i <= 2 and 1 <= j <= 2)] +
    [(1, i, j) for i in range(2, 6) for j in range(2, 6) if not (3 <= i <= 4 and 3 <= j <= 4)] +
    [(2, i, j) for i in range(6, 10) for j in range(6, 10)])


def _recursion(ctx, h, bufs, reg, t0, dt0):
    F, mask = h.finest(), 0

    def advance(l, t, dt, layer):
        nonlocal mask
        cur = (mask >> l) & 1
        mask ^= 1 << l
        ctx.patch_step(bufs[cur], bufs[cur ^ 1], *h.level_range(l), l, dt, layer, reg, h.side_mask_ptr(),
                       leaf_xy=h.leaf_xy_ptr(), t=t)
        if l < F:
            advance(l + 1, t, 0.5 * dt, 1)
            ctx.ghost_fill(h, bufs, mask, l + 1, l + 1)
            advance(l + 1, t + 0.5 * dt, 0.5 * dt, 0)
            ctx.flux_correct(h, bufs, mask, l, reg)

    for k in range(2):
        ctx.ghost_fill(h, bufs, mask, 0, 0)
        advance(0, t0 + k * dt0, dt0, 0)
    return mask


@pytest.mark.parametrize("prec", [af.FP64, af.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("m,tile", [(8, 8), (16, 8), (16, 16), (32, 4), (32, 8), (64, 2), (64, 4), (128, 2)])
@pytest.mark.parametrize("eq", ["rotation", "swirl", "burgers"])
def test_batched_equals_recursion(eq, m, tile, prec):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    kw = {"rotation": dict(eq=af.ROTATION, x0=-1.0, y0=-1.0, lx=2.0, ly=2.0, omega=1.0),
          "swirl": dict(eq=af.SWIRL), "burgers": dict(eq=af.BURGERS, qmax=1.0)}[eq]
    for leaves in (TWO, THREE):
        P = af.Problem(prec=prec, m=m, n0x=N0, n0y=N0, lmax=2, **kw)
        ctx = af.Context(P)
        ctx.tile = tile
        h = af.Hierarchy(ctx, leaves)
        rng = np.random.default_rng(m)
        blocks = [{k: rng.uniform(0.2, 0.6, (1, m + 5, m + 5)) for k in KINDS} for _ in leaves]
        start = af.blocks_to_state(ctx, blocks)
        s0 = [start, torch.zeros_like(start)]
        ctx.ghost_fill(h, s0, 0, 0, 0)
        t0, dt0 = 0.2, 0.4 * P.dx(0) / (1.5 if eq == "rotation" else 1.0)
        closed = closed_masks(m)

        def run(step):
            bufs = [s0[0].clone(), s0[1].clone()]
            reg = torch.zeros((len(leaves), 4, m, 1), dtype=torch.float64, device="cuda")
            mask = step(bufs, reg)
            torch.cuda.synchronize()
            assert float(reg.abs().max()) == 0.0
            g = [af.state_to_blocks(ctx, b) for b in bufs]
            return [g[(mask >> l) & 1][k] for k, (l, _, _) in enumerate(leaves)]

        def single(graph):
            def step(bufs, reg):
                mask = 0
                for k in range(2):
                    mask = ctx.amr_coarse_step(h, bufs, mask, dt0, reg, use_graph=graph, t0=t0 + k * dt0)
                return mask
            return step

        ref = run(lambda bufs, reg: _recursion(ctx, h, bufs, reg, t0, dt0))
        got = {}
        for fused in (True, False):
            ctx.fused_pairs = fused
            got[fused, "eager"] = run(single(False))
            got[fused, "graph"] = run(single(True))
            got[fused, "one call"] = run(
                lambda bufs, reg: ctx.amr_coarse_steps(h, bufs, 0, dt0, 2, reg, t0=t0))
        # a foot is known to a few roundings of its position (FP64: positions of
        # size 1, or 8 m N0 cells at most; FP32: of its displacement), a value
        # moves by about 4 per cell, in 8 substeps that amplify 3 times at most
        eps = 2.0 ** -53 * 16 * m * N0 if prec == af.FP64 else 2.0 ** -24 * 4 * 4
        for key, out in got.items():
            err = max(np.abs(out[i][k][0][closed[k]] - ref[i][k][0][closed[k]]).max()
                      for i in range(len(leaves)) for k in KINDS)
            assert err <= 4 * 8 * 3 * eps, (key, len(leaves), err)
