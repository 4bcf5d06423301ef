"""The one-sample-per-block tagger kernels at the edges of their shapes: input
channel counts around the padded widths 8, 16, 24, 32, a single sample, and
more samples than blocks.  Reference: FP64 convolutions (torch, CPU) of the
GPU's own BF16 operands, layer by layer, entry by entry:
|err| <= sqrt(K) 2^-24 sum |products| over the K terms of an entry."""
import os

import numpy as np
import pytest

import paper_2205_07572_amd as af

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


@pytest.mark.parametrize("nin,B", [(1, 1), (8, 3), (9, 2), (16, 1), (20, 2), (32, 3), (13, 257)])
def test_shapes(nin, B):
    torch = pytest.importorskip("torch")
    if not os.path.exists("/dev/kfd"):
        pytest.skip("no GPU on this machine")
    from torch.nn.functional import conv2d
    from torch.nn.grad import conv2d_input, conv2d_weight
    rng = np.random.default_rng(100 * nin + B)
    t = af.Tagger(nin)
    p = (0.25 * rng.standard_normal(t.nparams)).astype(np.float32)
    t.set_params(p)
    x = torch.from_numpy(rng.standard_normal((B, nin, 16, 16)).astype(np.float32))
    lab = torch.from_numpy(rng.integers(0, 3, B).astype(np.int32))
    grad = torch.full((t.nparams,), float("nan"), dtype=torch.float32, device="cuda")
    logits, acts = t.forward(x.cuda(), acts=True)
    loss, dacts = t.loss_grad(x.cuda(), lab.cuda(), grad, dacts=True)
    torch.cuda.synchronize()
    grad = grad.cpu().double()
    nchw = lambda a: a.cpu().double().reshape(3, B, 16, 16, 32).permute(0, 1, 4, 2, 3)  # noqa: E731
    z, da = nchw(acts), nchw(dacts)
    bf = lambda a: a.float().bfloat16().double()  # noqa: E731

    def check(name, got, ref, bound):
        ratio = ((got - ref).abs() / (bound + 1e-30)).max().item()
        assert ratio <= 1.0, (name, ratio)

    o, inp = 0, x.double()
    P = torch.from_numpy(p).double()
    for l, cin in enumerate((nin, 32, 32)):
        W, b = P[o:o + 288 * cin].reshape(32, cin, 3, 3), P[o + 288 * cin:o + 288 * cin + 32]
        gW, gb = grad[o:o + 288 * cin].reshape(W.shape), grad[o + 288 * cin:o + 288 * cin + 32]
        o += 288 * cin + 32
        a, w = bf(inp), bf(W)
        ref = conv2d(a, w, b, padding=1)
        mag = conv2d(a.abs(), w.abs(), b.abs(), padding=1)
        check(f"z{l}", z[l], ref, np.sqrt(9 * cin + 1) * U32 * mag)
        dz = torch.where(z[l] > 0, da[l], torch.zeros_like(da[l]))
        g, K = bf(dz), B * 256
        check(f"W{l}", gW, conv2d_weight(a, W.shape, g, padding=1),
              np.sqrt(K) * U32 * conv2d_weight(a.abs(), W.shape, g.abs(), padding=1))
        check(f"b{l}", gb, dz.sum(dim=(0, 2, 3)), np.sqrt(K) * U32 * dz.abs().sum(dim=(0, 2, 3)))
        if l:
            check(f"dA{l}", da[l - 1], conv2d_input(a.shape, w, g, padding=1),
                  np.sqrt(288 + 9) * U32 * conv2d_input(a.shape, w.abs(), g.abs(), padding=1))
        inp = z[l].clamp_min(0)
    # head: 256-term pooled sums, 32-term logits, a softmax of FP32 functions
    Wh, bh = P[o:o + 96].reshape(3, 32), P[o + 96:o + 99]
    pooled = inp.mean(dim=(2, 3))
    L = pooled @ Wh.T + bh
    tol = 512 * U32
    check("logits", logits.cpu().double(), L, tol * (pooled @ Wh.abs().T + bh.abs()))
    q = torch.softmax(L, 1) - torch.nn.functional.one_hot(lab.long(), 3)
    ref = -torch.log_softmax(L, 1)[torch.arange(B), lab.long()].mean()
    check("loss", loss.cpu().double(), ref[None], tol * (L.abs().max() + 1))
    check("Wh", grad[o:o + 96].reshape(3, 32), q.T @ pooled / B, tol * (L.abs().max() + 1) * pooled.sum(0)[None] / B)
    check("bh", grad[o + 96:o + 99], q.mean(0), tol * (L.abs().max() + 1))
