"""A batch, or a fit context, that has not run yet reports no status and no samples
outside the grid, whatever its workspace held before."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pairs", [1, 17, 40])
def test_nothing_to_report_before_the_first_run(gpu_lib, n_pairs):
    import torch
    S = gpu_lib
    n_sub, p, grid = 8, 6, 64
    n = n_sub * p
    pupil = wl.pupil_mask(n, float(n))
    valid = wl.valid_subapertures(pupil, p)
    wfs = S.Wfs.from_numpy(pupil, p, valid, device="cuda:0")
    F = torch.randn((n_pairs, grid, grid), device="cuda")
    stacks = [F[i:i + 1] for i in range(n_pairs)]
    pairs = [(0, i, S.affine_from_misreg((0.1 * (i % 3), 0.0, 0.01, 1.0), grid, grid, n, n)[0])
             for i in range(n_pairs)]

    def dirty():   # what the allocator hands out next holds ones
        torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device="cuda")

    torch.cuda.empty_cache()
    dirty()
    B = S.Batch([wfs], stacks, pairs)
    assert B.status() == 0 and B.oob() == 0
    B.run()
    assert B.status() == 0 and B.oob() == 0
    one = S.im_build(F[:1], pairs[0][2], wfs)
    assert (B.outs[0] - one).abs().max() <= 1e-5 * one.abs().max()
    torch.cuda.empty_cache()
    dirty()
    m = S.Misreg(wfs, F, np.array([-2, -2, -0.02, 0.98]), np.array([2, 2, 0.02, 1.02]),
                 max_batch=n_pairs, gn_batched=True)
    assert m.status() == 0
