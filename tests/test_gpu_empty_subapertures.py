"""Valid subapertures whose weights are all zero, whole tiles of them: no pixel of theirs
is in the pupil, or the edge repair leaves none of their samples.  Their slopes are 0 and
are written like all others, whatever the output held; the others match the oracle within
the parity tests' bounds, 1e-5 of the IM's and 1e-4 of a derivative plane's largest entry."""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim, repair as orep, tsum as ots

pytestmark = pytest.mark.gpu


def problem(S, n_sub, p, grid, n_act, disk):
    """A pupil disk around the centre, every subaperture listed as valid."""
    n = n_sub * p
    pupil = wl.pupil_mask(n, float(disk))
    valid = np.arange(n_sub * n_sub, dtype=np.int32)
    theta = (0.4, -0.7, 0.3, 1.05)
    A, dA = S.affine_from_misreg(theta, grid, grid, n, n)
    F = np.random.default_rng(n).standard_normal((n_act, grid, grid)).astype(np.float32)
    lit = pupil.reshape(n_sub, p, n_sub, p).sum(axis=(1, 3)).ravel() > 0
    return pupil, valid, theta, A, dA, F, lit


def check(got, ref, lit, tol):
    got = got.cpu().numpy()
    both = np.concatenate([lit, lit])
    assert 0 < lit.sum() < lit.size
    assert np.max(np.abs(got[:, both] - ref)) <= tol * np.abs(ref).max()
    assert np.all(got[:, ~both] == 0)


def dirty(shape):
    """What the allocator hands out next for this shape holds 777s."""
    import torch
    torch.full(shape, 777.0, device="cuda")


@pytest.mark.parametrize("n_sub,p,n_act,disk", [
    (24, 6, 70, 30), (40, 4, 9, 20), (25, 1, 130, 5), (12, 12, 33, 24)])
def test_no_pupil_pixel(gpu_lib, n_sub, p, n_act, disk):
    import torch
    S = gpu_lib
    grid = n_sub * p + 15
    pupil, valid, theta, A, dA, F, lit = problem(S, n_sub, p, grid, n_act, disk)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    Fd = torch.from_numpy(F).cuda()
    args = (F, A[:, :2], A[:, 2], pupil, p, valid[lit])
    ref, tref = oim.im_build(*args), ots.im_build_tsum(*args)
    Jref = oim.jacobian(F, theta, pupil, p, valid[lit])
    shape = (n_act, 2 * len(valid))
    out = torch.full(shape, 777.0, device="cuda")
    check(S.im_build(Fd, A, wfs, out=out), ref, lit, 1e-5)
    out.fill_(777.0)
    check(S.im_build_tsum(Fd, A, wfs, out=out), tref, lit, 1e-5)
    dirty((4,) + shape)
    dirty(shape)
    im, J = S.im_jacobian(Fd, A, dA, wfs)
    check(im, ref, lit, 1e-5)
    for j in range(4):
        check(J[j], Jref[j], lit, 1e-4)
    other = S.Wfs.from_numpy(pupil, p, valid[lit], device="cuda:0")
    for sensors in ([wfs], [wfs, wfs], [wfs, other]):
        B = S.Batch(sensors, [Fd], [(i, 0, A) for i in range(len(sensors))])
        for o in B.outs:
            o.fill_(777.0)
        B.run()
        torch.cuda.synchronize()
        for w, o in zip(sensors, B.outs):
            if w is wfs:
                check(o, ref, lit, 1e-5)
            else:
                assert np.max(np.abs(o.cpu().numpy() - ref)) <= 1e-5 * np.abs(ref).max()
        B.close()


@pytest.mark.parametrize("n_sub,p,n_act,core", [(24, 6, 70, 40), (25, 1, 130, 9), (26, 4, 3, 30)])
def test_nothing_left_by_the_repair(gpu_lib, n_sub, p, n_act, core):
    import torch
    S = gpu_lib
    n = n_sub * p
    grid = n + 7
    pupil, valid, theta, A, dA, F, _ = problem(S, n_sub, p, grid, n_act, 2 * n)
    M = wl.pupil_mask(grid, float(core)).astype(np.uint8)
    F = F * M
    ref = orep.im_build_repaired(F, M, A[:, :2], A[:, 2], pupil, p, valid)
    assert (np.abs(ref).max(axis=0) == 0).any()
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    out = torch.full((n_act, 2 * len(valid)), 777.0, device="cuda")
    got = S.im_build_repaired(torch.from_numpy(F).cuda(), torch.from_numpy(M).cuda(), A, wfs,
                              out=out).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.abs(ref).max()


def test_every_configuration(gpu_lib):
    import torch
    S = gpu_lib
    n_sub, p, grid = 8, 10, 96
    pupil, valid, _, A, _, F, lit = problem(S, n_sub, p, grid, 40, 20)
    A, _ = S.affine_from_misreg((0.2, -0.3, 0.01, 1.0), grid, grid, 80, 80)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    ref = oim.im_build(F, A[:, :2], A[:, 2], pupil, p, valid[lit])
    Fd = torch.from_numpy(F).cuda()
    cands = S.im_candidates(wfs, A)
    assert any(c["schedule"] != 0 for c in cands)
    for c in cands:
        S.im_set_config(wfs, A, c)
        ws = S.im_plan(wfs, A, device=Fd.device)
        out = torch.full((40, 2 * len(valid)), 777.0, device="cuda")
        check(S.im_apply(Fd, A, wfs, ws, out=out), ref, lit, 1e-5)
    S.autotune_clear()
