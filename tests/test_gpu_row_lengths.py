"""IF rows of every length modulo 4, at any 4-byte address, in every call that
streams them: the sensor well inside the grid (16-byte DMA), against its right
edge and beyond (the row's last, partial vector is staged), turned by half and by
a quarter.  Against the oracle with the parity tests' bounds: 1e-5 of the largest
element of the IM, 1e-4 of that of a derivative plane.
"""
import math

import numpy as np
import pytest

import workloads as wl
from oracle import im as oim, repair as orep

pytestmark = pytest.mark.gpu


def stack(n, H, W, offset, seed=3):
    """Random IFs on the device at `offset` floats from an allocation's start."""
    import torch
    F = np.random.default_rng(seed).standard_normal((n, H, W)).astype(np.float32)
    flat = torch.empty(F.size + offset, dtype=torch.float32, device="cuda")
    flat[offset:] = torch.from_numpy(F.ravel()).cuda()
    return F, flat[offset:].view(n, H, W)


CASES = [
    (61, 0, (0.3, -0.2, 0.02, 1.0)),
    (62, 1, (0.3, -0.2, 0.3, 1.0)),
    (63, 2, (-0.3, 0.4, math.pi, 1.0)),
    (63, 3, (0.2, 0.1, math.pi / 2 + 0.01, 0.98)),
    (61, 3, (6.7, 0.2, 0.01, 1.0)),       # the last columns
    (62, 0, (-7.3, 0.2, math.pi, 1.02)),
    (63, 1, (15.5, 3.2, 0.1, 1.0)),       # beyond the grid
    (64, 1, (0.3, -0.2, 0.02, 1.0)),      # whole vectors at an odd address
]


@pytest.mark.parametrize("W,offset,theta", CASES)
def test_row_lengths(gpu_lib, W, offset, theta):
    import torch
    S = gpu_lib
    p, n = 6, 48
    pupil = wl.pupil_mask(n, float(n), 0.2)
    valid = wl.valid_subapertures(pupil, p)
    F, dev = stack(9, 62, W, offset)
    A, dA = S.affine_from_misreg(theta, 62, W, n, n)
    wfs = S.Wfs.from_numpy(pupil, p, valid)
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid)
    tol = 1e-5 * np.abs(ref).max()
    assert np.max(np.abs(S.im_build(dev, A, wfs).cpu().numpy() - ref)) <= tol
    ws = S.im_plan(wfs, A)
    assert np.max(np.abs(S.im_apply(dev, A, wfs, ws).cpu().numpy() - ref)) <= tol
    im, J = S.im_jacobian(dev, A, dA, wfs)
    assert np.max(np.abs(im.cpu().numpy() - ref)) <= tol
    Jref = oim.jacobian(F, theta, pupil, p, valid)
    J = J.cpu().numpy()
    for j in range(4):
        assert np.max(np.abs(J[j] - Jref[j])) <= 1e-4 * np.abs(Jref[j]).max()
    w = np.random.default_rng(1).standard_normal(ref.shape).astype(np.float32)
    grad = S.im_vjp(dev, A, dA, wfs, torch.from_numpy(w).cuda()).cpu().numpy()
    for j in range(4):
        assert abs(grad[j] - np.sum(w * Jref[j])) <= 1e-4 * np.sum(np.abs(w * Jref[j]))
    mask = np.zeros((62, W), np.uint8)
    mask[2:-2, 2:-2] = 1
    M = F * mask
    got = S.im_build_repaired(torch.from_numpy(M).cuda(), torch.from_numpy(mask).cuda(), A,
                              wfs).cpu().numpy()
    rr = orep.im_build_repaired(M, mask, A[:, :2], A[:, 2], pupil, p, valid, 0.999999)
    assert np.max(np.abs(got - rr)) <= 1e-5 * np.abs(rr).max()
