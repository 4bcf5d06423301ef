"""Layouts past the edge of 32-bit arithmetic: more leaves than one launch of
four blocks of 256 threads per leaf can take (a grid holds 2^32 threads)."""
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
