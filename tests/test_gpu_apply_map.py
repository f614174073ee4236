"""A plan streams the rows of the map it was built for: the map a later im_apply
names only picks the kernel configuration, by its linear part.

On grids of every row length, planned against the right edge and beyond it (where a
row's last, partial 16-byte vector is staged) and applied with a map shifted to the
middle, and the other way round: the oracle's IM of the planned map, to the parity
tests' 1e-5 of its largest element.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import im as oim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [61, 62, 63, 64])
@pytest.mark.parametrize("planned,named", [(6.7, -6.0), (9.4, 0.0), (-6.0, 6.7)])
def test_planned_map_is_streamed(gpu_lib, W, planned, named):
    import torch
    S = gpu_lib
    p, n = 6, 48
    pupil = wl.pupil_mask(n, float(n), 0.2)
    valid = wl.valid_subapertures(pupil, p)
    F = np.random.default_rng(7).standard_normal((9, 62, W)).astype(np.float32)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    maps = [S.affine_from_misreg((-t, 0.2, 0.01, 1.0), 62, W, n, n)[0] for t in (planned, named)]
    ws = S.im_plan(wfs, maps[0])
    got = S.im_apply(torch.from_numpy(F).cuda(), maps[1], wfs, ws).cpu().numpy()
    ref = oim.im_build(F, maps[0][:, :2], maps[0][:, 2], pupil, p, valid)
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.abs(ref).max()
