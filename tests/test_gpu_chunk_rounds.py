"""Launches of several rounds with few chunks: eight or sixteen chunks in the queues of
all XCDs where two to fifteen would fill the workgroups evenly, stacks of fewer
actuators than queues.  IM and derivative planes against the FP64 oracle with the
parity tests' bounds, 1e-5 of the IM's and 1e-4 of a plane's largest entry; launches
on one plan repeat bit for bit (the queues' counters end at zero); the VJP is the
sum of the library's own derivative planes in FP64, in another order.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sub,n_act,rot", [
    (80, 3, 0.008),      # fewer chunks than queues
    (80, 70, 0.008),
    (80, 150, 0.008),
    (64, 40, 0.4),
    (110, 45, 0.008),
    (110, 330, 0.008),   # several rounds of the IM alone
])
def test_few_chunks(gpu_lib, n_sub, n_act, rot):
    import torch
    S = gpu_lib
    p = 2
    n = n_sub * p
    pupil = wl.pupil_mask(n, float(n))
    valid = wl.valid_subapertures(pupil, p)
    grid = n + 16
    F = np.random.default_rng(3).standard_normal((n_act, grid, grid)).astype(np.float32)
    theta = (0.3, -0.2, rot, 1.01)
    A, dA = S.affine_from_misreg(theta, grid, grid, n, n)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    Fd = torch.from_numpy(F).cuda()
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid)
    ws = S.im_plan(wfs, A, dA, planes=5)
    first = S.im_apply(Fd, A, wfs, ws, planes=5)
    assert np.max(np.abs(first.cpu().numpy() - ref)) <= 1e-5 * np.abs(ref).max()
    for _ in range(3):
        assert torch.equal(S.im_apply(Fd, A, wfs, ws, planes=5), first)
    im, dim = S.im_jacobian(Fd, A, dA, wfs, ws=ws)
    assert torch.equal(im, first)
    for j in range(4):
        assert torch.equal(S.im_apply(Fd, A, wfs, ws, planes=5, plane=1 + j), dim[j])
    few = slice(0, n_act, max(1, n_act // 8))
    J = oim.jacobian(F[few], theta, pupil, p, valid)
    for j in range(4):
        d = dim[j].cpu().numpy()[few]
        assert np.max(np.abs(d - J[j])) <= 1e-4 * np.abs(J[j]).max()
    g = torch.randn(ref.shape, generator=torch.Generator().manual_seed(4)).cuda()
    terms = dim.double() * g.double()[None]
    want, scale = terms.sum(dim=(1, 2)), terms.abs().sum(dim=(1, 2))
    for _ in range(3):
        assert torch.all((S.im_vjp(Fd, A, dA, wfs, g, ws=None) - want).abs() <= 1e-12 * scale)
