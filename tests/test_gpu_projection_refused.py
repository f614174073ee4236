"""Systems that are not positive definite are refused by their status word, wherever
the pivot that shows it falls: a function that is zero everywhere, without a
regularisation, in each kind of place the factorisation has (the first column of all,
another of the first 16, a later group of 16, a later block of 64, a later panel of
256, the last column); values that are not finite; and the same functions with a
regularisation, which the oracle's P_opt answers to the solves' 1e-9."""
import numpy as np
import pytest

import workloads as wl
from oracle import projection as opj

pytestmark = pytest.mark.gpu

DIRS = np.array([[0.0, 0.0], [2e-4, -1e-4]])
E_PARAM = -3


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def functions(n, grid, width, seed):
    """Gaussians at different grid points under the pupil."""
    y, x = np.mgrid[0:grid, 0:grid]
    c = np.argwhere(np.hypot(x - (grid - 1) / 2, y - (grid - 1) / 2) <= 17)
    c = c[np.random.default_rng(seed).choice(len(c), n, replace=False)]
    d2 = (x - c[:, 1, None, None]) ** 2 + (y - c[:, 0, None, None]) ** 2
    return np.exp(-d2 / (2 * width ** 2)).astype(np.float32)


@pytest.mark.parametrize("at", [0, 5, 20, 70, 300, 319])
def test_zero_function(gpu_lib, at):
    S = gpu_lib
    pupil = wl.pupil_mask(40, 40.0)
    F, G = functions(320, 48, 0.5, 1), functions(20, 48, 5.0, 2)
    layers = [(dev(G), 3000.0, 0.5)]
    # as they are, the functions are independent: lambda = 0 is accepted
    S.proj_opt([(dev(F), 0.0, 0.5)], layers, DIRS, pupil, 0.5, 0.0)
    F[at] = 0
    with pytest.raises(S.SynimError) as e:
        S.proj_opt([(dev(F), 0.0, 0.5)], layers, DIRS, pupil, 0.5, 0.0)
    assert e.value.status == E_PARAM
    P_dm = opj.projection_matrix([(F, 0.0, 0.5)], DIRS, pupil, 0.5, 1)
    P_l = opj.projection_matrix([(G, 3000.0, 0.5)], DIRS, pupil, 0.5, 1)
    lam = 1e-2 * np.trace(P_dm.T @ P_dm) / 320
    ref = opj.p_opt(P_dm, P_l, lam)
    got = S.proj_opt([(dev(F), 0.0, 0.5)], layers, DIRS, pupil, 0.5, lam).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-9 * np.abs(ref).max()
    assert np.all(got[at] == 0)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("at", [3, 66, 301])
def test_not_finite(gpu_lib, bad, at):
    S = gpu_lib
    pupil = wl.pupil_mask(40, 40.0)
    F = functions(320, 48, 0.5, 1)
    F[at, 24, 24] = bad
    layers = [(dev(functions(20, 48, 5.0, 2)), 3000.0, 0.5)]
    with pytest.raises(S.SynimError) as e:
        S.proj_opt([(dev(F), 0.0, 0.5)], layers, DIRS, pupil, 0.5, 1.0)
    assert e.value.status == E_PARAM
