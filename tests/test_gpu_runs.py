"""The warp kernel's runs of influence functions against the oracle: counts on both
sides of a run of eight, of the six runs from which each XCD takes its own, and of
whole eights of runs.  The bound is the parity tests': 1e-6 of the largest sample
(four rounded products)."""
import numpy as np
import pytest

from oracle import warp as owarp

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
