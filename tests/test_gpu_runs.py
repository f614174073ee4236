"""The warp and slope kernels' runs of maps and forms by pixels per subaperture,
against the oracle.

Warp: counts on both sides of a run of eight, of the six runs from which each XCD
takes its own, and of whole eights of runs.  Slopes: every form the pixels of a
subaperture pick (whole rows of loads, and ones that are left out), groups of one,
two and four subaperture rows, one map a run to eight.  The bounds are those of the
parity tests: 1e-6 of the largest sample for the warp (four rounded products),
1e-5 of the largest slope (sums of rounded differences)."""
import numpy as np
import pytest

import workloads as wl
from oracle import slopes as osl, warp as owarp

pytestmark = pytest.mark.gpu


def to_dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n", [1, 2, 8, 9, 17, 40, 41, 48, 63, 64, 65, 130])
def test_warp_runs(gpu_lib, n):
    F = np.random.default_rng(n).standard_normal((n, 60, 61)).astype(np.float32)
    A, _ = gpu_lib.affine_from_misreg((0.3, -0.2, 0.05, 1.01), 60, 61, 41, 47)
    got = gpu_lib.affine_warp(to_dev(F), A, 41, 47, halo=1).cpu().numpy()
    ref = owarp.warp(F, A[:, :2], A[:, 2], 41, 47, 1)
    assert got.shape == ref.shape
    assert np.max(np.abs(got - ref)) <= 1e-6 * np.abs(F).max()


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 13, 16, 20, 25, 28, 32, 33, 49, 64])
@pytest.mark.parametrize("n_sub,n", [(1, 1), (3, 9), (5, 47)])
def test_slope_forms(gpu_lib, p, n_sub, n):
    size = n_sub * p
    pupil = wl.pupil_mask(size, float(size) if p > 2 else 2.0 * size, 0.3 if n_sub > 3 else 0.0)
    valid = wl.valid_subapertures(pupil, p)
    phase = np.random.default_rng(size).standard_normal((n, size + 2, size + 2)).astype(np.float32)
    got = gpu_lib.sa_slopes(to_dev(phase), gpu_lib.Wfs.from_numpy(pupil, p, valid)).cpu().numpy()
    ref = osl.slopes(phase, pupil, p, valid)
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.max(np.abs(ref))


@pytest.mark.parametrize("n_sub,p,n", [
    (60, 6, 17),       # one row a group, several maps a run
    (60, 6, 150),      # two rows
    (90, 2, 400),      # four rows, the last group short
    (91, 5, 130),      # an odd number of rows in groups of four
])
def test_slope_runs(gpu_lib, n_sub, p, n):
    import torch
    size = n_sub * p
    pupil = wl.pupil_mask(size, float(size), 0.2)
    valid = wl.valid_subapertures(pupil, p)
    few = np.random.default_rng(size).standard_normal((7, size + 2, size + 2)).astype(np.float32)
    ref = osl.slopes(few, pupil, p, valid)
    wfs = gpu_lib.Wfs.from_numpy(pupil, p, valid)
    which = torch.arange(n) % 7
    got = gpu_lib.sa_slopes(to_dev(few)[which.cuda()].contiguous(), wfs)
    alone = gpu_lib.sa_slopes(to_dev(few), wfs)
    assert torch.equal(got, alone[which.cuda()])   # whatever the run and the group
    assert np.max(np.abs(alone.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
