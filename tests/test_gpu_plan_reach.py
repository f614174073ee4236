"""Maps that shrink one axis of the WFS grid into one IF cell: their inverses reach
over more pixels than a 32-bit integer counts, and every sample still has its weight.

Along the shrunk axis neighbouring samples lie 2.5e-10 IF pixels apart near
coordinate 10, where FP64 coordinates carry roundings of 9e-16: their differences
are known to 4e-6 in the library and in the oracle alike, sums over a subaperture's
pixels no worse, and the patch weights are rounded to FP32 once.  1e-4 of that axis'
largest slope leaves room for both; the other axis keeps the parity tests' 1e-5.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [4, 8, 10, 21])   # with and without the table of samples
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("a", [2.5e-10, -2.5e-10])
def test_axis_in_one_cell(gpu_lib, p, axis, a):
    import torch
    S = gpu_lib
    n = 4 * p
    pupil = wl.pupil_mask(n, float(n))
    valid = wl.valid_subapertures(pupil, p)
    F = np.random.default_rng(2).standard_normal((3, 24, 24)).astype(np.float32)
    A = np.array([[0.2, 0.0, 3.3], [0.0, 0.2, 2.7]])
    A[axis] = [0.0, 0.0, 10.25]
    A[axis, axis] = a
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid).reshape(3, 2, -1)
    tol = np.array([1e-5, 1e-5])
    tol[axis] = 1e-4
    tol = (tol * np.abs(ref).max(axis=(0, 2)))[None, :, None]
    Fd = torch.from_numpy(F).cuda()
    got = S.im_build(Fd, A, wfs).cpu().numpy().reshape(ref.shape)
    assert np.all(np.abs(got - ref) <= tol)
    dA = np.zeros((4, 2, 3))
    dA[0, 0, 2] = dA[1, 1, 2] = -1.0
    im, _ = S.im_jacobian(Fd, A, dA, wfs)
    assert np.all(np.abs(im.cpu().numpy().reshape(ref.shape) - ref) <= tol)
