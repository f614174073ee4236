"""The plan at the edges of its launch shapes, against the oracle: several small
subapertures per workgroup and one with more patch entries than threads, pupil
masks that fit 64 bits and ones that do not, sensors of one subaperture and of
rows longer than a wave, quarter and half turns (each sign of the map's linear
part), windows that leave the IF grid, valid subapertures without a neighbour.
Bounds as in the parity tests: 1e-5 of the largest element; counts are equal.
"""
import math

import numpy as np
import pytest

import workloads as wl
from oracle import im as oim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sub,p,grid,theta,keep", [
    (5, 2, 24, (0.2, 0.1, 0.05, 1.0), 1),
    (70, 2, 160, (0.2, -0.3, 0.3, 0.97), 1),       # more than 64 subapertures a row
    (1, 8, 24, (0.2, 0.1, 0.1, 1.0), 1),           # one subaperture
    (6, 8, 60, (0.1, 0.2, math.pi / 2, 1.0), 1),
    (6, 9, 66, (0.1, 0.2, -math.pi / 2 + 0.02, 1.02), 1),   # 81 pixels a subaperture
    (4, 13, 64, (0.3, 0.2, math.pi + 0.01, 0.99), 1),       # over 256 patch entries
    (12, 5, 64, (7.4, -6.3, 0.4, 1.03), 3),        # leaves the grid; every third kept
])
def test_plan_forms(gpu_lib, n_sub, p, grid, theta, keep):
    import torch
    n = n_sub * p
    pupil = wl.pupil_mask(n, float(n) * (1.0 if n_sub > 1 else 2.0), 0.15 if n_sub > 4 else 0.0)
    valid = wl.valid_subapertures(pupil, p)[::keep].copy()
    F = np.random.default_rng(n).standard_normal((5, grid, grid)).astype(np.float32)
    A, _ = gpu_lib.affine_from_misreg(theta, grid, grid, n, n)
    wfs = gpu_lib.Wfs.from_numpy(pupil, p, valid)
    ws = gpu_lib.im_plan(wfs, A, grid=(grid, grid))
    assert gpu_lib.plan_status(ws) == 0
    assert gpu_lib.plan_oob(ws) == oim.oob_count(A[:, :2], A[:, 2], pupil, p, valid, grid, grid)
    got = gpu_lib.im_apply(torch.from_numpy(F).cuda(), A, wfs, ws).cpu().numpy()
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid)
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.abs(ref).max()
