"""The warp and slope kernels at the edges of their launch shapes, against the oracle.

Warp: fewer and more influence functions than the eight of one pass, windows
narrower and wider than a workgroup and of an odd width, maps whose taps leave
the grid.  Slopes: subapertures of one pixel, more pixel rows per group than a
thread keeps as bits (64), odd grids, grids of several workgroups, runs of maps
that do not divide the batch.  The bounds are those of the parity tests: 1e-6 of
the largest sample for the warp (four rounded products), 1e-5 of the largest
slope (sums of rounded differences).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import slopes as osl, warp as owarp

pytestmark = pytest.mark.gpu


def to_dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n,Hi,Wi,H,W,halo,theta", [
    (1, 40, 41, 37, 39, 1, (0.3, -0.2, 0.02, 1.01)),
    (7, 64, 64, 33, 127, 0, (0.5, 0.25, 0.01, 0.98)),
    (9, 140, 300, 120, 255, 1, (0.4, 0.1, 0.03, 1.02)),
    (61, 70, 71, 65, 65, 1, (0.37, -0.81, 0.12, 1.03)),
    (130, 160, 160, 150, 131, 2, (60.5, -33.25, 0.3, 0.9)),   # many taps off the grid
    (517, 128, 128, 118, 118, 1, (0.2, 0.1, 0.05, 1.0)),      # runs of eight, the last short
])
def test_warp_forms(gpu_lib, n, Hi, Wi, H, W, halo, theta):
    import torch
    F = np.random.default_rng(n).standard_normal((n, Hi, Wi)).astype(np.float32)
    A, _ = gpu_lib.affine_from_misreg(theta, Hi, Wi, H, W)
    oob = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = gpu_lib.affine_warp(to_dev(F), A, H, W, halo=halo, oob=oob).cpu().numpy()
    ref, n_oob = owarp.warp(F, A[:, :2], A[:, 2], H, W, halo, count_oob=True)
    assert np.max(np.abs(got - ref)) <= 1e-6 * np.abs(F).max()
    assert int(oob.item()) == n_oob


@pytest.mark.parametrize("n_sub,p,n", [
    (33, 1, 3),       # one pixel per subaperture
    (21, 2, 5),
    (9, 7, 70),       # odd grid: the last column has no right neighbour of its own
    (11, 9, 11),      # 72 pixel rows per group: pupil read per row
    (5, 64, 2),       # the widest subaperture
    (90, 6, 9),       # more columns than a workgroup
    (3, 5, 1500),     # short runs of many maps
])
def test_slopes_forms(gpu_lib, n_sub, p, n):
    size = n_sub * p
    pupil = wl.pupil_mask(size, float(size), 0.2)
    valid = wl.valid_subapertures(pupil, p)
    phase = np.random.default_rng(size).standard_normal((n, size + 2, size + 2)).astype(np.float32)
    got = gpu_lib.sa_slopes(to_dev(phase), gpu_lib.Wfs.from_numpy(pupil, p, valid)).cpu().numpy()
    ref = osl.slopes(phase, pupil, p, valid)
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.max(np.abs(ref))


@pytest.mark.parametrize("n_sub,p,n", [
    (9, 3, 3600),     # two subaperture rows a workgroup, the last group one
    (9, 3, 5600),     # four
    (6, 12, 8300),    # four of 12 pixels, the last group two
    (5, 17, 8300),    # 68 pixel rows: pupil read per row
])
def test_slopes_rows_per_workgroup(gpu_lib, n_sub, p, n):
    import torch
    size = n_sub * p
    pupil = wl.pupil_mask(size, float(size), 0.2)
    valid = wl.valid_subapertures(pupil, p)
    base = np.random.default_rng(size).standard_normal((61, size + 2, size + 2)).astype(np.float32)
    at = np.arange(n) % 61
    phase = to_dev(base)[torch.from_numpy(at).cuda()]
    got = gpu_lib.sa_slopes(phase, gpu_lib.Wfs.from_numpy(pupil, p, valid)).cpu().numpy()
    ref = osl.slopes(base, pupil, p, valid)
    assert np.max(np.abs(got - ref[at])) <= 1e-5 * np.max(np.abs(ref))
