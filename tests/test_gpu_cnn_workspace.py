"""One call of a tagger entry point makes the workspace of all: the others, up
to the same number of samples, can then be captured into a graph (nothing is
allocated in the capture) and replay the eager results."""
import os

import numpy as np
import pytest

import afsynth
import paper_2205_07572_amd as af

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("warm", ["forward", "loss_grad", "tag"])
def test_captured_after_another_call(warm):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    B, m = 16, 16
    rng = np.random.default_rng(3)
    P = af.Problem(eq=af.ACOUSTICS, prec=af.FP32, m=m, n0x=4, n0y=4, lmax=1, c=1.0)
    ctx = af.Context(P)
    h = af.Hierarchy(ctx, afsynth.uniform_leaves(4, 4, 0))
    h.leaf_xy_ptr()  # the hierarchy's tables are on the device
    state = ctx.new_state(B)
    state.uniform_(-1.0, 1.0)
    plain = torch.zeros(B, dtype=torch.int8, device="cuda")
    x = torch.from_numpy(rng.standard_normal((B, 13, m, m)).astype(np.float32)).cuda()
    lab = torch.from_numpy(rng.integers(0, 3, B).astype(np.int32)).cuda()
    p = (0.25 * rng.standard_normal(af.Tagger(13).nparams)).astype(np.float32)

    def calls(t):
        grad = torch.zeros(t.nparams, dtype=torch.float32, device="cuda")
        return {"forward": lambda: t.forward(x), "loss_grad": lambda: (t.loss_grad(x, lab, grad), grad)[1],
                "tag": lambda: t.tag(ctx, h, [state, state], 0, plain)[1]}

    ref = af.Tagger(13)
    ref.set_params(p)
    want = {k: f().clone() for k, f in calls(ref).items()}
    for name in want:
        t = af.Tagger(13)
        t.set_params(p)
        c = calls(t)
        c[warm]()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            out = c[name]()
        for _ in range(2):
            out.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want[name]), (warm, name)
