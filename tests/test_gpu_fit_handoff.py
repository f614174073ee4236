"""Samples of a large batch that a Gauss-Newton fit leaves to later launches.

Six of the ten samples used here hop between bilinear cells past the first
launch's iterations.  With up to 12 such samples in a batch each is split over
workgroups, with more they go on in one workgroup each.  Either way an estimate
is a function of the batch alone: it repeats bit for bit, with and without a graph,
and does not depend on where in the batch its sample stands.
"""
import pytest

pytestmark = pytest.mark.gpu
DRAWS = [1000269, 1000577, 1000812, 1000895, 1000957, 1000978, 7, 8, 9, 10]


def _fit(S, copies):
    from paper_2606_07759_amd import learned
    sy = learned.probe_system("cuda")
    theta, snr, noise = learned.draw(DRAWS, sy.M)
    m = S.Misreg(sy.wfs, sy.probes, sy.lo, sy.hi, max_batch=10 * copies)
    one = learned.synthesize(m, theta, snr, noise, 10)
    return m, one.repeat(copies, 1).contiguous()


@pytest.mark.parametrize("copies", [1, 2, 3, 4])   # 6, 12, 18, 24 slow samples
def test_estimates_repeat(gpu_lib, copies):
    import torch
    m, s = _fit(gpu_lib, copies)
    a, ia = m.infer(s, use_graph=False)
    bad = m.unconverged()
    assert bad == int((ia >= 20).sum().item()) and int((ia > 10).sum().item()) == 6 * copies
    out = (torch.empty_like(a), torch.empty_like(ia))
    for k in range(12):
        if k % 3 == 0:
            b, ib = m.infer(s, use_graph=False)
        else:
            b, ib = m.infer(s, out=out)
        assert torch.equal(b, a) and torch.equal(ib, ia) and m.unconverged() == bad
    # equal samples, equal bits, wherever they stand
    for r in range(1, copies):
        assert torch.equal(a[10 * r:10 * r + 10], a[:10])
        assert torch.equal(ia[10 * r:10 * r + 10], ia[:10])
    perm = torch.randperm(10 * copies, generator=torch.Generator().manual_seed(1)).cuda()
    b, ib = m.infer(s[perm].contiguous(), use_graph=False)
    assert torch.equal(b, a[perm]) and torch.equal(ib, ia[perm])


@pytest.mark.parametrize("copies", [1, 2])
def test_workgroups_that_stop_waiting(gpu_lib, copies):
    """Split samples whose workgroups give up waiting for each other (after one poll)
    are finished in one workgroup: the same iterations, the same count of
    unconverged samples, estimates within the 1e-6 the two forms' orders of
    summation leave between samples that hop."""
    import torch
    S = gpu_lib
    m, s = _fit(S, copies)
    a, ia = m.infer(s, use_graph=False)
    bad = m.unconverged()
    lib = S.load()
    assert lib.synim_misreg_set_polls(None, 1) == -1
    assert lib.synim_misreg_set_polls(m._h, 0) == -3
    assert lib.synim_misreg_set_polls(m._h, 1) == 0
    out = (torch.empty_like(a), torch.empty_like(ia))
    for graph in (False, True, True):
        b, ib = m.infer(s, use_graph=graph, out=out)
        torch.cuda.synchronize()
        assert torch.equal(ib, ia) and m.unconverged() == bad
        assert (b - a).abs().max().item() <= 1e-6


@pytest.mark.parametrize("L,xc,steps", [(2.3, -30.0, 16), (3.0, -36.0, 13)])
@pytest.mark.parametrize("batch,late", [(4, 3), (12, 8), (20, 16)])   # split, split after, one workgroup
def test_steps_of_a_sample_that_turns_singular(gpu_lib, L, xc, steps, batch, late):
    """Measured slopes of zero on probes that fall off as exp(x / L): every step moves
    the sensor by L down the exponential, until it has left the probes, which are zero
    there, and the normal matrix is singular.  The steps taken until then are the
    oracle's (the same with its slopes and derivatives rounded to FP32); a sample
    that stops so is not converged."""
    import numpy as np
    import torch
    from oracle import im as oim
    S = gpu_lib
    n_sub, p, grid = 2, 4, 128
    y, x = np.mgrid[0:grid, 0:grid] - (grid - 1) / 2.0
    e = np.exp((x - 4.0) / L) * (x > xc)
    probes = np.stack([e, e * np.sin(y / 3.0), e * np.cos(y / 2.0)]).astype(np.float32)
    pupil, valid = np.ones((8, 8), np.uint8), np.arange(4)
    lo, hi = np.array([-45, -4, -0.02, 0.98]), np.array([45, 4, 0.02, 1.02])
    span = hi - lo
    th, taken = np.array([0.0, 0.0, 0.0, 1.0]), 0
    F = probes.astype(np.float64)
    while taken < 40:
        s = oim.im_build_misreg(F, th, pupil, p, valid).ravel()
        J = oim.jacobian(F, th, pupil, p, valid).reshape(4, -1).T
        try:
            np.linalg.cholesky(J.T @ J)
        except np.linalg.LinAlgError:
            break
        th = np.clip(th + np.linalg.solve(J.T @ J, -J.T @ s), lo - 0.5 * span, hi + 0.5 * span)
        taken += 1
    assert taken == steps
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    m = S.Misreg(wfs, torch.from_numpy(probes).cuda(), lo, hi, max_batch=batch, max_iter=40)
    near = torch.tensor([[0.4, 0.2, 0.003, 1.002]], dtype=torch.float64, device="cuda")
    meas = m.slopes(near.repeat(batch, 1))
    meas[:late] = 0
    zero = (meas == 0).all(dim=1)
    assert int(zero.sum()) == late
    for graph in (False, True, True, True):
        _, it = m.infer(meas, use_graph=graph)
        assert torch.all(it[zero] == steps), it[zero].tolist()
        assert torch.all((it[~zero] > 0) & (it[~zero] <= 10))
        assert m.unconverged() == late
