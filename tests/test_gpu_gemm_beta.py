"""FP64 products with and without the old C: without (beta = 0) C's values are never
read, also where they are not finite; an empty sum scales C.  Against FP64 products on
the host: K products of rounding 1.1e-16 each stay within 1e-14 of their magnitudes'
sum for K <= 64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (64, 64, 64), (129, 130, 17), (200, 3, 33), (128, 128, 0)])
@pytest.mark.parametrize("beta", [0.0, 1.0, -0.5])
def test_beta(gpu_lib, M, N, K, beta):
    import torch
    rng = np.random.default_rng(M + N + K)
    X, Y = rng.standard_normal((max(K, 1), M)), rng.standard_normal((max(K, 1), N))
    C0 = rng.standard_normal((M, N))
    C = torch.from_numpy(C0.copy()).cuda()
    if beta == 0.0:
        C.fill_(float("nan"))
        C[0, 0] = float("inf")
    gpu_lib.gemm_f64(M, N, K, 2.0, torch.from_numpy(X).cuda(), M, 1, torch.from_numpy(Y).cuda(), N, 1,
                     beta, C, N)
    ref = 2.0 * X[:K].T @ Y[:K] + (beta * C0 if beta else 0.0)
    tol = 1e-14 * (2.0 * np.abs(X[:K]).T @ np.abs(Y[:K]) + abs(beta) * np.abs(C0) + 1e-300)
    assert np.all(np.abs(C.cpu().numpy() - ref) <= tol)
