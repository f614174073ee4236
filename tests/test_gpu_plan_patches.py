"""The largest weight patches (24 x 20 and 24 x 24 entries, more than the threads of the
smaller ones' workgroups) in every build that plans them, on few subapertures and on
many: against the oracle with the parity tests' bounds, 1e-5 of the IM's and 1e-4 of a
derivative plane's largest entry."""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim, tsum as ots

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sub,p,rot,patch", [
    (2, 10, 0.6, (24, 20)),
    (8, 10, 0.78, (24, 20)),
    (5, 13, 0.6, (24, 24)),
    (3, 21, 0.02, (24, 24)),      # more samples than the plan's table holds
])
def test_large_patches(gpu_lib, n_sub, p, rot, patch):
    import torch
    S = gpu_lib
    n = n_sub * p
    grid = int(1.45 * n) + 12
    pupil = wl.pupil_mask(n, 1.2 * n)
    valid = wl.valid_subapertures(pupil, p)
    theta = (0.2, -0.3, rot, 1.0 if p < 20 else 1.08)
    A, dA = S.affine_from_misreg(theta, grid, grid, n, n)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    cfg = S.im_config(wfs, A)
    assert (cfg["patch_rows"], cfg["patch_cols"]) == patch
    F = np.random.default_rng(n).standard_normal((6, grid, grid)).astype(np.float32)
    Fd = torch.from_numpy(F).cuda()
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid)
    im, J = S.im_jacobian(Fd, A, dA, wfs)
    for got in (S.im_build(Fd, A, wfs), im):
        assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-5 * np.abs(ref).max()
    Jref = oim.jacobian(F, theta, pupil, p, valid)
    for j in range(4):
        assert np.max(np.abs(J[j].cpu().numpy() - Jref[j])) <= 1e-4 * np.abs(Jref[j]).max()
    ts = S.im_build_tsum(Fd, A, wfs).cpu().numpy()
    tref = ots.im_build_tsum(F, A[:, :2], A[:, 2], pupil, p, valid)
    assert np.max(np.abs(ts - tref)) <= 1e-5 * np.abs(tref).max()
