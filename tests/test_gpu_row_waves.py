"""One and four waves a block row: solves and Lanczos runs on both sides of the lines
where the launches change over, for blocks of 4 and 6 and short and long rows,
against a sparse LU."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spl

from test_gpu_shared_rows import chain

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1002_1202_amd import api
    assert torch.cuda.is_available()
    return api.Context(0)


def system(ctx, nb, B, reach):
    from paper_1002_1202_amd import api
    rowptr, colidx, H, S = chain(np.random.default_rng(nb + B), nb, B, reach)
    pair = api.Pair(ctx, B, rowptr, colidx, H=H, S=S)
    return pair, *(sp.bsr_array((V, colidx, rowptr), shape=(nb * B, nb * B)).tocsc() for V in (S, H))


# Chebyshev steps: one chunk, complex64 from 4096 block rows, FP64 from 12288; seed
# product by rows times chunks
@pytest.mark.parametrize("nb,B,R,reach,precision",
                         [(4095, 4, 64, (0, 1, 2), "mixed"), (4096, 4, 64, (0, 1, 2), "mixed"),
                          (4096, 4, 192, (0, 1), "mixed"), (4097, 6, 7, (1,), "mixed"),
                          (12287, 4, 3, (0, 2), "fp64"), (12288, 4, 64, (0, 1), "fp64"),
                          (12289, 6, 2, (0, 1), "fp64"), (12289, 6, 2, (0, 1), "mixed"),
                          (2048, 4, 250, (0, 2), "fp64"), (1366, 6, 322, (1, 2), "fp64"),
                          (2731, 6, 130, (9, 10), "fp64"), (4096, 6, 64, (9, 10), "mixed")])
def test_solve_vs_lu(ctx, nb, B, R, reach, precision):
    from paper_1002_1202_amd import api
    print(f"case: waves nb={nb} B={B} R={R} reach={reach} {precision}", flush=True)
    pair, S, H = system(ctx, nb, B, reach)
    N = nb * B
    rhs = np.sort(np.random.default_rng(R).choice(N, size=R, replace=False)).astype(np.int64)
    z = np.array([-3 + 0.5j, 1 + 0.5j])
    res = api.solve(ctx, pair, z, rhs=rhs, tol=1e-12, precision=precision)
    assert res.status == 0 and res.converged.all()
    E = np.zeros((N, R), complex)
    E[rhs, np.arange(R)] = 1.0
    for k, zk in enumerate(z):
        # |x - x_k| <= |A^-1| tol: A's smallest singular value is at least Im z
        # times S's smallest eigenvalue (0.6 by its rows), with a factor of ten
        X = spl.splu((zk * S - H).tocsc()).solve(E)
        assert np.linalg.norm(res.G_cols[k].T - X, axis=0).max() <= 10 * 1e-12 / (0.5 * 0.6)


# two processes a column
@pytest.mark.parametrize("nb,B,P,reach", [(2047, 4, 256, (0, 2)), (2048, 4, 256, (0, 2)), (2048, 4, 509, (0, 1)),
                                          (1365, 6, 770, (1,)), (1366, 6, 770, (1,)), (1366, 6, 700, (9, 10))])
def test_lanczos_vs_lu(ctx, nb, B, P, reach):
    from paper_1002_1202_amd import api
    print(f"case: waves Lanczos nb={nb} B={B} P={P} reach={reach}", flush=True)
    pair, S, H = system(ctx, nb, B, reach)
    N = nb * B
    rhs = np.sort(np.random.default_rng(P).choice(N, size=P, replace=False)).astype(np.int64)
    z = np.array([-2 + 2j, 1 + 2j])
    res = api.lanczos_green(ctx, pair, z, rhs, tol=1e-12)
    E = np.zeros((N, P), complex)
    E[rhs, np.arange(P)] = 1.0
    for k, zk in enumerate(z):
        G = spl.splu((zk * S - H).tocsc()).solve(E)[rhs, np.arange(P)]
        # ended when 16 further steps change G by at most 1e-12 of its largest; with
        # Im z S of at least 1.2 against |H| of at most 100 they shrink the error by
        # exp(-32 asinh(1.2 / 100)) = 0.68, so 2.1e-12 are left, with a factor of ten
        assert np.abs(res.G_diag[k] - G).max() <= 2.2e-11 * np.abs(G).max()
