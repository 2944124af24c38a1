"""The inner CG's product on both sides of the line where it gives a short block row
one wave instead of four, and with long rows, against a sparse LU."""
import numpy as np
import pytest
import scipy.sparse.linalg as spl

from test_gpu_row_waves import system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,B,R,reach", [(4095, 4, 3, (0, 1)), (4096, 4, 64, (0, 1)), (2049, 4, 66, (0, 2)),
                                          (4097, 6, 5, (0, 1)), (500, 6, 70, (9, 10))])
def test_cg_solve_vs_lu(nb, B, R, reach):
    import torch
    from paper_1002_1202_amd import api
    assert torch.cuda.is_available()
    print(f"case: CG waves nb={nb} B={B} R={R} reach={reach}", flush=True)
    pair, S, H = system(api.Context(0), nb, B, reach)
    N = nb * B
    rhs = np.sort(np.random.default_rng(R).choice(N, size=R, replace=False)).astype(np.int64)
    z = np.array([-3 + 0.5j, 1 + 0.5j])
    res = api.solve(pair.ctx, pair, z, rhs=rhs, tol=1e-12, inner_method=1)
    assert res.status == 0 and res.converged.all()
    E = np.zeros((N, R), complex)
    E[rhs, np.arange(R)] = 1.0
    for k, zk in enumerate(z):
        # |x - x_k| <= |A^-1| tol: A's smallest singular value is at least Im z
        # times S's smallest eigenvalue (0.6 by its rows), with a factor of ten
        X = spl.splu((zk * S - H).tocsc()).solve(E)
        assert np.linalg.norm(res.G_cols[k].T - X, axis=0).max() <= 10 * 1e-12 / (0.5 * 0.6)
