"""The direct FP32 products at the edges of their tiles, steps and column maps.

Widths in whole float4 (what the direct products take) that are no multiples of
the 16- and 32-wide tiles or of the 32-deep steps, one to eight outputs, batches
of a few rows past the small-batch path up to several tiles, segments that touch
and that leave gaps, and odd shapes next to them that take the staged products.
FP32 sums of at most 2080 products against the FP64 oracle: 1e-4 of the largest
entry, as for the estimator's own shape.
"""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,h1,h2,n_out,segs,B", [
    (212, 36, 20, 1, ((4, 60), (100, 44)), 17),
    (212, 36, 20, 8, ((4, 60), (64, 148)), 33),     # segments that touch
    (64, 4, 4, 3, ((0, 4), (60, 4)), 20),           # smallest widths
    (2048, 512, 64, 4, ((0, 32), (1000, 1028)), 600),
    (512, 160, 132, 5, ((0, 0), (8, 96)), 1200),    # one segment, 32 x 32 tiles
    (212, 36, 20, 4, ((4, 60), (101, 44)), 33),     # staged: a segment off by one
    (212, 34, 20, 9, ((4, 60), (100, 44)), 33),     # staged: width, outputs
])
def test_direct_products(gpu_lib, n_in, h1, h2, n_out, segs, B):
    import torch
    S = gpu_lib
    net = S.Mlp(n_in, h1, h2, n_out, segs)
    rng = np.random.default_rng(B)
    shapes = [(h1, n_in), (h1,), (h2, h1), (h2,), (n_out, h2), (n_out,)]
    parts = [(rng.standard_normal(s) * (2.0 / s[-1]) ** 0.5).astype(np.float32) for s in shapes]
    (s0, l0), (s1, l1) = segs
    xc = rng.standard_normal((B, l0 + l1)).astype(np.float32)
    t = rng.uniform(-1, 1, (B, n_out)).astype(np.float32)
    params = torch.from_numpy(np.concatenate([p.ravel() for p in parts])).cuda()
    xd, td = torch.from_numpy(xc).cuda(), torch.from_numpy(t).cuda()
    scratch = net.scratch(B)
    y = net.forward(params, xd, scratch)
    grads = torch.full_like(params, float("nan"))   # fully overwritten
    loss = torch.zeros(1, device="cuda")
    net.backward(params, xd, scratch, y, td, grads, loss)
    x = np.zeros((B, n_in))
    x[:, s0:s0 + l0] = xc[:, :l0]
    x[:, s1:s1 + l1] = xc[:, l0:]
    P = [p.astype(np.float64) for p in parts]
    yref, acts = omlp.forward(x, [(P[0], P[1]), (P[2], P[3]), (P[4], P[5])])

    def err(got, ref):
        return float(np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30))
    assert err(y.cpu().numpy(), yref) <= 1e-4
    assert abs(loss.item() - omlp.mse(yref, t)) <= 1e-4 * omlp.mse(yref, t)
    gref = omlp.backward(acts, [(P[0], P[1]), (P[2], P[3]), (P[4], P[5])], t.astype(np.float64))
    g = grads.cpu().numpy()
    for (lo, hi), ref in zip(net.layout(), [a for pair in gref for a in pair]):
        assert err(g[lo:hi].reshape(ref.shape), ref) <= 1e-4, (lo, hi)
    W1 = g[:h1 * n_in].reshape(h1, n_in)
    used = np.zeros(n_in, bool)
    used[s0:s0 + l0] = used[s1:s1 + l1] = True
    assert np.all(W1[:, ~used] == 0)
    g2 = torch.empty_like(grads)
    net.backward(params, xd, scratch, y, td, g2)
    assert torch.equal(g2, grads)
