"""The two-level factorisation and solves at block and panel edges (64 and 256
columns), right-hand sides on both sides of a workgroup's 32, against the FP64
oracle with the parity test's bound (1e-9 of the largest element of P_opt); a
system whose matrix is not finite is refused."""
import numpy as np
import pytest

import workloads as wl
from oracle import projection as opj

pytestmark = pytest.mark.gpu

DIRS = np.array([[0.0, 0.0], [2e-4, -1e-4]])


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def functions(n, grid, width, seed):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:grid, 0:grid]
    c = rng.uniform(0, grid - 1, (n, 2))
    d2 = (x - c[:, 0, None, None]) ** 2 + (y - c[:, 1, None, None]) ** 2
    return np.exp(-d2 / (2 * width ** 2)).astype(np.float32)


@pytest.mark.parametrize("n_dm,n_l", [(1, 1), (63, 33), (64, 32), (65, 31), (256, 5), (257, 64),
                                      (321, 40), (520, 17)])
def test_panels(gpu_lib, n_dm, n_l):
    pupil = wl.pupil_mask(40, 40.0, 0.2)
    dms = [(functions(n_dm, 48, 2.0, 1), 0.0, 0.5)]
    layers = [(functions(n_l, 48, 5.0, 2), 3000.0, 0.5)]
    P_dm = opj.projection_matrix(dms, DIRS, pupil, 0.5, 1)
    P_l = opj.projection_matrix(layers, DIRS, pupil, 0.5, 1)
    lam = 1e-2 * np.trace(P_dm.T @ P_dm) / P_dm.shape[1]
    ref = opj.p_opt(P_dm, P_l, lam)
    got = gpu_lib.proj_opt([(dev(F), h, s) for F, h, s in dms], [(dev(F), h, s) for F, h, s in layers],
                           DIRS, pupil, 0.5, lam).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-9 * np.abs(ref).max()


def test_not_finite_refused(gpu_lib):
    pupil = wl.pupil_mask(40, 40.0, 0.2)
    F = functions(70, 48, 2.0, 1)
    F[66, 24, 12] = np.nan
    dms = [(dev(F), 0.0, 0.5)]
    layers = [(dev(functions(20, 48, 5.0, 2)), 3000.0, 0.5)]
    with pytest.raises(Exception):
        gpu_lib.proj_opt(dms, layers, DIRS, pupil, 0.5, 1.0)
