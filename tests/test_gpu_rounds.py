"""Item counts at the edges of the stream kernel's work distribution.

A launch whose items all fit one round of workgroups touches no counter (with
chunks that are, or are not, a multiple of the 8 XCDs); a larger one hands the
rest out by counters that it leaves zero for the next launch on the same plan;
waves whose slots are all empty do no contraction.  Each against the FP64
oracle: FP32 products of weights rounded once, summed in at most 256 terms, stay
within 1e-5 of the largest entry.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim

pytestmark = pytest.mark.gpu
IM_TOL = 1e-5


def _case(n_sub, p, n_act, seed=3):
    n = n_sub * p
    pupil = wl.pupil_mask(n, float(n))
    valid = wl.valid_subapertures(pupil, p)
    F = np.random.default_rng(seed).standard_normal((n_act, n + 16, n + 16)).astype(np.float32)
    return F, pupil, valid


@pytest.mark.parametrize("n_sub,p,n_act", [
    (8, 10, 1), (8, 10, 3), (8, 10, 9), (8, 10, 64), (8, 10, 300),   # one round
    (5, 4, 33),                                                       # tiles mostly empty
    (40, 2, 1100),                                                    # several rounds
])
def test_rounds(gpu_lib, n_sub, p, n_act):
    import torch
    S = gpu_lib
    F, pupil, valid = _case(n_sub, p, n_act)
    n = n_sub * p
    A, dA = S.affine_from_misreg((0.3, -0.2, 0.008, 1.01), n + 16, n + 16, n, n)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    Fd = torch.from_numpy(F).cuda()
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid)
    ws = S.im_plan(wfs, A, device="cuda:0", grid=(n + 16, n + 16))
    outs = [S.im_apply(Fd, A, wfs, ws).cpu().numpy() for _ in range(3)]   # one plan, three launches
    for got in outs:
        assert np.max(np.abs(got - ref)) <= IM_TOL * np.max(np.abs(ref))
        assert np.array_equal(got, outs[0])
    if n_act <= 64:
        g = torch.from_numpy(np.random.default_rng(4).standard_normal(ref.shape).astype(np.float32)).cuda()
        _, dim = S.im_jacobian(Fd, A, dA, wfs)
        want = (dim.double() * g.double()[None]).sum(dim=(1, 2)).cpu().numpy()
        got = S.im_vjp(Fd, A, dA, wfs, g).cpu().numpy()
        # the same FP32 slopes, summed in FP64 in another order
        scale = (dim.double().abs() * g.double().abs()[None]).sum(dim=(1, 2)).cpu().numpy()
        assert np.all(np.abs(got - want) <= 1e-12 * scale)
