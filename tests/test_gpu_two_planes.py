"""Derivative planes in pairs: every (block, lanes, rows, columns) the ranking can
pick over pixel sizes and turns, chunk counts below, at and above a round, and
grids that keep the one-plane kernel (rows no multiple of 4 whose last vector is
staged).  Against the oracle with the parity test's bound, 1e-4 of the largest
element of each plane.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sub,p,grid,n,theta", [
    (6, 4, 32, 1, (0.3, -0.2, 0.02, 1.0)),
    (12, 5, 72, 7, (0.3, -0.2, 0.3, 1.02)),
    (20, 6, 136, 40, (0.3, -0.2, 0.02, 1.0)),
    (16, 7, 128, 130, (-0.4, 0.2, 0.7, 0.97)),
    (9, 10, 104, 17, (0.1, 0.4, 0.01, 1.0)),
    (5, 16, 100, 9, (0.1, 0.4, 0.2, 1.05)),
    (12, 5, 61, 9, (0.3, -0.2, 0.02, 1.0)),
])
def test_pairs_of_planes(gpu_lib, n_sub, p, grid, n, theta):
    import torch
    size = n_sub * p
    pupil = wl.pupil_mask(size, float(size), 0.2)
    valid = wl.valid_subapertures(pupil, p)
    F = np.random.default_rng(n).standard_normal((n, grid, grid)).astype(np.float32)
    A, dA = gpu_lib.affine_from_misreg(theta, grid, grid, size, size)
    wfs = gpu_lib.Wfs.from_numpy(pupil, p, valid)
    dev = torch.from_numpy(F).cuda()
    im, J = gpu_lib.im_jacobian(dev, A, dA, wfs)
    ref = oim.jacobian(F, theta, pupil, p, valid)
    J = J.cpu().numpy()
    for j in range(4):
        assert np.max(np.abs(J[j] - ref[j])) <= 1e-4 * np.abs(ref[j]).max()
    # the pairs' planes are the single planes, bit for bit
    ws = gpu_lib.im_plan(wfs, A, dA=dA, planes=5)
    for j in range(4):
        assert np.array_equal(gpu_lib.im_apply(dev, A, wfs, ws, planes=5, plane=1 + j).cpu().numpy(),
                              J[j])
