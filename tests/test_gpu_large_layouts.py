"""Layouts past the edge of 32-bit arithmetic: more leaves than one launch of
four blocks of 256 threads per leaf, or one of 1024, can take (a grid holds less
than 2^32 threads), and a row pitch that makes the plane of one patch larger than 4 GiB."""
import os

import numpy as np
import pytest

import afsynth
import paper_2205_07572_amd as af

pytestmark = pytest.mark.gpu


def _need(bytes_):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    if torch.cuda.mem_get_info()[0] < bytes_ + (8 << 30):
        pytest.skip("not enough device memory")
    return torch


@pytest.mark.parametrize("call", ["patch_step", "coarse_step", "level_advance"])
@pytest.mark.parametrize("eq,m", [(af.ADVECTION, 8), (af.BURGERS, 8), (af.ACOUSTICS, 16)])
def test_wide_rows(eq, m, call):
    if call == "level_advance" and (eq == af.BURGERS or m == 8):
        pytest.skip("no level-advance kernel for it")
    P = af.Problem(eq=eq, prec=af.FP32, m=m, a=1.0, b=0.5, c=1.0, qmax=1.0)
    S = m + 5
    wide = (1 << 30) // (m + 1) + 1  # elements: the last rows that a step writes begin past 2^32 bytes
    torch = _need(2 * 4 * P.ncomp * S * wide * 4)
    ctx = af.Context(P)
    h = af.Hierarchy(ctx, afsynth.uniform_leaves(1, 1, 0))
    rng = np.random.default_rng(2)
    # periodic data on one patch: the high lines and ghost layers repeat the interior
    core = torch.from_numpy(rng.uniform(0.2, 0.6, (4, P.ncomp, 1, m, m)).astype(np.float32)).cuda()
    idx = (torch.arange(S, device="cuda") - 2) % m
    block = core[..., idx, :][..., idx]
    out = []
    for pitch in (S, wide):
        bufs = [torch.empty((4, P.ncomp, 1, S, pitch), dtype=torch.float32, device="cuda") for _ in range(2)]
        for b in bufs:
            b[..., :S] = block
        dt = 0.4 * P.dx(0)
        if call == "patch_step":
            ctx.patch_step(bufs[0], bufs[1], 0, 1, 0, dt)
            mask = 1
        elif call == "coarse_step":
            reg = torch.zeros((1, 4, m, P.ncomp), dtype=torch.float64, device="cuda")
            mask = ctx.amr_coarse_step(h, bufs, 0, dt, reg)
        else:
            mask = ctx.level_advance(h, bufs, 0, 0, dt, 2)
        torch.cuda.synchronize()
        r = bufs[mask & 1][..., 2:3 + m, 2:3 + m].clone()
        r[0, ..., m, :] = r[0, ..., :, m] = r[2, ..., m, :] = r[3, ..., :, m] = 0  # entries that no step defines
        out.append(r)
        del bufs, b
        torch.cuda.empty_cache()
    # the same arithmetic, but the two layouts may take different kernels: each
    # of at most two steps sums up to 60 products of values below 1, 32 units
    # of rounding at most
    assert float((out[0] - out[1]).abs().max()) <= 64 * 2.0 ** -24
    assert float((out[0][1] - block[1, ..., 2:3 + m, 2:3 + m]).abs().max()) > 1e-3  # a step was made


def test_transfer_of_many_leaves():
    n0 = 2056  # 4.2 million leaves
    P = af.Problem(eq=af.ADVECTION, prec=af.FP32, m=8, n0x=n0, n0y=n0)
    torch = _need(2 * 4 * n0 * n0 * 13 * 13 * 4)
    ctx = af.Context(P)
    iy, ix = np.divmod(np.arange(n0 * n0), n0)
    leaves = np.stack([np.zeros_like(ix), ix, iy], 1)
    old, new = af.Hierarchy(ctx, leaves), af.Hierarchy(ctx, leaves)
    src = ctx.new_state(n0 * n0)
    src.uniform_(-1.0, 1.0)
    dst = ctx.new_state(n0 * n0)
    ctx.regrid_apply(old, [src, src], 0, new, dst)
    torch.cuda.synchronize()
    for k, (r, c) in enumerate(((8, 8), (9, 9), (8, 9), (9, 8))):
        assert torch.equal(src[k, :, :, 2:2 + r, 2:2 + c], dst[k, :, :, 2:2 + r, 2:2 + c]), k


def test_level_advance_of_many_patches():
    """A set block size whose grid would reach 2^32 threads is replaced."""
    n0, m = 2056, 16
    P = af.Problem(eq=af.ADVECTION, prec=af.FP32, m=m, n0x=n0, n0y=n0, lx=float(n0), ly=float(n0), a=1.0, b=0.5)
    torch = _need(4 * 4 * n0 * n0 * 21 * 21 * 4)
    iy, ix = np.divmod(np.arange(n0 * n0), n0)
    leaves = np.stack([np.zeros_like(ix), ix, iy], 1)
    ctx = af.Context(P)
    start = ctx.new_state(n0 * n0)
    start.uniform_(-1.0, 1.0)
    h = af.Hierarchy(ctx, leaves)
    out = []
    for shape in ((8, 256), (16, 1024)):
        ctx.set_advance_shape(*shape)
        bufs = [start.clone(), torch.zeros_like(start)]
        mask = ctx.level_advance(h, bufs, 0, 0, 0.4 * P.dx(0), 16)
        torch.cuda.synchronize()
        s = bufs[mask & 1][:, :, -4096:, 2:2 + m, 2:2 + m].clone()
        out.append(s)
        del bufs
        torch.cuda.empty_cache()
    # rounding of about 10 operations of weight 1 per step, in random order
    assert float((out[0] - out[1]).abs().max()) <= 16 * 16 * 2.0 ** -24
    assert float(out[0].abs().max()) > 0.1
