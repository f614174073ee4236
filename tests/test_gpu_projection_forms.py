"""The window sampler and the step-skipping products of the projection at their
edges, against the FP64 oracle.

Sampling: every window size (2, 4, 6, 8 grid points a side) and a block too wide
for the largest, pupil blocks cut by the mask, footprints that leave the grid,
function counts on both sides of a group and of a tile of 128 columns, and a
function with a value that is not finite: the samples that have it as a tap are
not finite, no other is.  Products: local functions (many empty steps), tiles
split into parts and not, odd row counts, a workspace that only holds the
matrices.  Bounds as in the parity tests of the same entry points: 1e-12 of the
largest sample, 1e-9 of the largest element of P_opt.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import projection as opj

pytestmark = pytest.mark.gpu


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def local_functions(n, grid, width, seed):
    """n Gaussians of the given width at random places, zero beyond 4 widths."""
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:grid, 0:grid]
    c = rng.uniform(0, grid - 1, (n, 2))
    d2 = (x - c[:, 0, None, None]) ** 2 + (y - c[:, 1, None, None]) ** 2
    return np.where(d2 < (4 * width) ** 2, np.exp(-d2 / (2 * width ** 2)), 0).astype(np.float32)


DIRS = np.array([[0.0, 0.0], [2e-4, -1e-4], [-1.5e-4, 2.5e-4]])


@pytest.mark.parametrize("b,scale,n", [
    (1, 1.0, 3),       # window 2
    (2, 1.0, 130),     # 4
    (3, 1.0, 70),      # 6, blocks of 3
    (4, 1.0, 9),       # 6: taps on grid points exactly, where rounding moves the cell
    (4, 0.61, 65),     # 8
    (4, 1.7, 16),      # several pixels in one cell
    (6, 0.8, 5),       # wider than the largest window
])
def test_sampler_windows(gpu_lib, b, scale, n):
    pupil = wl.pupil_mask(60, 57.0, 0.2)
    comps = [(local_functions(n, 64, 4.0, 1), 0.0, 0.5 * scale),
             (local_functions(n + 1, 53, 5.0, 2), 30000.0, 0.5 * scale)]   # leaves the grid
    got = gpu_lib.proj_matrix([(dev(F), h, s) for F, h, s in comps], DIRS, pupil, 0.5,
                              bin=b).cpu().numpy().T
    ref = opj.projection_matrix(comps, DIRS, pupil, 0.5, b)
    assert np.max(np.abs(got - ref)) <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_sampler_not_finite(gpu_lib, bad):
    pupil = wl.pupil_mask(40, 40.0)
    F = local_functions(10, 48, 4.0, 3)
    G = F.copy()
    G[4, 20, 23] = bad
    # pixel centres fall between grid points: a sample has four taps of its own
    args = (np.array([[0.25 * 0.5 / 9000.0, 0.1 * 0.5 / 9000.0]]), pupil, 0.5)
    got = gpu_lib.proj_matrix([(dev(G), 9000.0, 0.5)], *args, bin=2).cpu().numpy().T
    with np.errstate(invalid="ignore"):
        ref = opj.projection_matrix([(G, 9000.0, 0.5)], *args, 2)
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    assert 0 < np.count_nonzero(~np.isfinite(got)) < 10
    ok = np.isfinite(ref)
    assert np.max(np.abs(got[ok] - ref[ok])) <= 1e-12 * np.abs(ref[ok]).max()


@pytest.mark.parametrize("n_dm,n_l,size,b", [
    (40, 30, 48, 1),      # one tile, split into parts
    (129, 257, 90, 2),    # ragged tiles
    (300, 128, 63, 1),    # odd row count: pairs of rows at any 8-byte address
])
def test_popt_local(gpu_lib, n_dm, n_l, size, b):
    import torch
    pupil = wl.pupil_mask(size, float(size), 0.2)
    grid = size + 12
    dms = [(local_functions(n_dm // 2, grid, 3.0, 5), 0.0, 0.5),
           (local_functions(n_dm - n_dm // 2, grid, 4.0, 6), 4000.0, 0.5)]
    layers = [(local_functions(n_l, grid, 6.0, 7), 2000.0, 0.5)]
    P_dm = opj.projection_matrix(dms, DIRS, pupil, 0.5, b)
    P_l = opj.projection_matrix(layers, DIRS, pupil, 0.5, b)
    lam = 1e-2 * np.trace(P_dm.T @ P_dm) / P_dm.shape[1]
    ref = opj.p_opt(P_dm, P_l, lam)
    d = [(dev(F), h, s) for F, h, s in dms]
    l = [(dev(F), h, s) for F, h, s in layers]
    need = gpu_lib.proj_workspace_bytes(d, l, len(DIRS), pupil, bin=b)
    for nbytes in (need, need - 1):   # one byte less: the dense products
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        got = gpu_lib.proj_opt(d, l, DIRS, pupil, 0.5, lam, bin=b, ws=ws).cpu().numpy()
        assert np.max(np.abs(got - ref)) <= 1e-9 * np.abs(ref).max()
