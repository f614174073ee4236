"""P_opt of blocks wider than the largest sampling window, whose samples are formed
one by one: functions that are zero over most of the pupil and functions that are
zero nowhere, rows that do and do not fill a wave or a step of 16, against the FP64
oracle with the parity test's bound (1e-9 of the largest element)."""
import numpy as np
import pytest

import workloads as wl
from oracle import projection as opj

pytestmark = pytest.mark.gpu

DIRS = np.array([[0.0, 0.0], [2e-4, -1e-4], [-1.5e-4, 2.5e-4]])


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def functions(n, grid, width, seed, dense):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:grid, 0:grid]
    c = rng.uniform(0, grid - 1, (n, 2))
    d2 = (x - c[:, 0, None, None]) ** 2 + (y - c[:, 1, None, None]) ** 2
    f = np.where(d2 < (4 * width) ** 2, np.exp(-d2 / (2 * width ** 2)), 0)
    return (f + 0.1 * dense * rng.standard_normal(f.shape)).astype(np.float32)


@pytest.mark.parametrize("n_dm,n_l,size,b,dirs", [
    (20, 10, 40, 8, 1),       # fewer rows than a wave
    (130, 60, 96, 8, 3),
    (140, 129, 150, 6, 3),    # 6 x 6 pixels over 8 grid points and more
])
@pytest.mark.parametrize("dense", [0, 1])
def test_wide_blocks(gpu_lib, n_dm, n_l, size, b, dirs, dense):
    import torch
    pupil = wl.pupil_mask(size, float(size), 0.2)
    step = 0.5 if b == 8 else 0.3
    grid = int(size * 0.5 / step) + 12
    dms = [(functions(n_dm, grid, 3.0, 5, dense), 0.0, step)]
    layers = [(functions(n_l, grid, 6.0, 7, dense), 2000.0, step)]
    P_dm = opj.projection_matrix(dms, DIRS[:dirs], pupil, 0.5, b)
    P_l = opj.projection_matrix(layers, DIRS[:dirs], pupil, 0.5, b)
    lam = 1e-2 * np.trace(P_dm.T @ P_dm) / P_dm.shape[1]
    ref = opj.p_opt(P_dm, P_l, lam)
    d = [(dev(F), h, s) for F, h, s in dms]
    l = [(dev(F), h, s) for F, h, s in layers]
    need = gpu_lib.proj_workspace_bytes(d, l, dirs, pupil, bin=b)
    for nbytes in (need, need - 1):   # one byte less: the dense products
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        got = gpu_lib.proj_opt(d, l, DIRS[:dirs], pupil, 0.5, lam, bin=b, ws=ws).cpu().numpy()
        assert np.max(np.abs(got - ref)) <= 1e-9 * np.abs(ref).max()
