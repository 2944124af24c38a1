"""Full carry of many shifts on both sides of the line where small systems go from
one workgroup a column to the tiles."""
import numpy as np
import pytest

from test_gpu_small import system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,B,K", [(128, 4, 1280), (128, 4, 1281), (1, 4, 2048), (1, 4, 2049), (16, 6, 2048),
                                    (16, 6, 2049)])
def test_many_shifts_vs_dense(nb, B, K):
    import torch
    from paper_1002_1202_amd import api
    assert torch.cuda.is_available()
    print(f"case: small shifts nb={nb} B={B} K={K}", flush=True)
    ctx = api.Context(0)
    pair, H, S, _, _ = system(ctx, nb, B, (0, 1))
    N = nb * B
    rhs = np.array([0, N // 2, N - 1])
    z = np.linspace(-6, 6, K) + 0.3j
    res = api.solve(ctx, pair, z, rhs=rhs, tol=1e-12)
    assert res.status == 0 and res.converged.all()
    L = np.linalg.inv(np.linalg.cholesky(S))
    lam, V = np.linalg.eigh(L @ H @ L.T)
    C = L.T @ V
    X = (1.0 / (z[:, None] - lam))[:, None, :] * C[rhs] @ C.T
    # |x - x_k| <= |A^-1| tol: A's smallest singular value is at least Im z times
    # S's smallest eigenvalue (0.6 by its rows), with a factor of ten
    assert np.linalg.norm(res.G_cols - X, axis=2).max() <= 10 * 1e-12 / (0.3 * 0.6)
