"""The forms of the one-launch Gauss-Newton kernel agree with the batched fit.

Batch sizes on both sides of the split over workgroups (8), a batch with samples
slow enough for the second launch, sensors whose points fit the registers (N <=
64, at most 80 points each) and sensors that do not, and probe planes that do
and do not fit the two region buffers.  The batched path (gn_batched) forms the
same normal equations from planned weight patches: both stop when the normalised
step is below 1e-6, so converged estimates agree to that step's scale.
"""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _system(n_sub, p, grid, n_probe, seed=5):
    n = n_sub * p
    pupil = wl.pupil_mask(n, float(n))
    valid = wl.valid_subapertures(pupil, p)
    c = (grid - 1) / 2.0
    y, x = (np.mgrid[0:grid, 0:grid] - c) / (n / 2.0)
    rng = np.random.default_rng(seed)
    probes = sum(rng.standard_normal((n_probe, 1, 1)) * x ** a * y ** b
                 for a in range(4) for b in range(4 - a))
    return probes.astype(np.float32), pupil, valid


@pytest.mark.parametrize("n_sub,p,grid,n_probe,batch", [
    (8, 10, 128, 20, 1),      # whole plane per workgroup
    (8, 10, 128, 20, 8),
    (8, 10, 128, 20, 9),      # one workgroup per sample
    (8, 10, 104, 3, 5),       # regions that reach outside the grid
    (8, 10, 200, 4, 3),       # plane larger than the region buffers
    (10, 8, 120, 5, 2),       # 80 subapertures: coordinates formed per probe
    (10, 8, 120, 5, 12),
    (4, 18, 91, 2, 2),        # more than 80 points, rows of an odd length
])
def test_forms_agree(gpu_lib, n_sub, p, grid, n_probe, batch):
    import torch
    S = gpu_lib
    probes, pupil, valid = _system(n_sub, p, grid, n_probe)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    pr = torch.from_numpy(probes).cuda()
    lo, hi = np.array([-4, -4, -0.02, 0.98]), np.array([4, 4, 0.02, 1.02])
    th = np.random.default_rng(6).uniform(0.7 * lo + 0.3 * hi, 0.3 * lo + 0.7 * hi, (batch, 4))
    one = S.Misreg(wfs, pr, lo, hi, max_batch=batch)
    many = S.Misreg(wfs, pr, lo, hi, max_batch=batch, gn_batched=True)
    s = one.slopes(torch.from_numpy(th).cuda())
    a, ia = one.infer(s, use_graph=False)
    b, ib = many.infer(s, use_graph=False)
    d = (a - b).abs().cpu().numpy() / (0.5 * (hi - lo))
    ok = (ia.cpu().numpy() < 20) & (ib.cpu().numpy() < 20)
    assert ok.mean() >= 0.9 and ia.min().item() >= 0
    assert d[ok].max() <= 2e-6
    assert one.unconverged() == int((ia.cpu().numpy() >= 20).sum())


def test_slow_samples_match_smaller_batches(gpu_lib):
    """Samples that run past the first launch's iterations end where a batch small
    enough to be split from the start ends, graph or no graph."""
    import torch
    from paper_2606_07759_amd import learned
    sy = learned.probe_system("cuda")
    theta, snr, noise = learned.draw([1000269, 1000577, 1000812, 1000895, 1000957, 1000978, 7, 8, 9, 10], sy.M)
    S = gpu_lib
    big = S.Misreg(sy.wfs, sy.probes, sy.lo, sy.hi, max_batch=40)
    s = learned.synthesize(big, theta, snr, noise, 10)
    s40 = s.repeat(4, 1).contiguous()   # 24 slow samples: more than the list holds
    a, ia = big.infer(s40, use_graph=False)
    n_bad = big.unconverged()
    small = S.Misreg(sy.wfs, sy.probes, sy.lo, sy.hi, max_batch=5)
    for k in (0, 5):
        b, ib = small.infer(s[k:k + 5].contiguous(), use_graph=False)
        for r in range(4):
            assert torch.equal(ia[10 * r + k:10 * r + k + 5], ib)
            assert (a[10 * r + k:10 * r + k + 5] - b).abs().max().item() <= 1e-6
    assert n_bad == int((ia >= 20).sum().item()) and n_bad >= 12
    out = (torch.empty_like(a), torch.empty_like(ia))
    for _ in range(3):
        big.infer(s40, out=out)
        assert torch.equal(out[1], ia) and big.unconverged() == n_bad
