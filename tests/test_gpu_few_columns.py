"""Products of tiles with few columns at work: a column's values do not depend on
which others are there, and solves of one to nine columns match a sparse LU."""
import numpy as np
import pytest
import scipy.sparse.linalg as spl

from test_gpu_row_waves import system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1002_1202_amd import api
    assert torch.cuda.is_available()
    return api.Context(0)


@pytest.mark.parametrize("nb,B,reach", [(33, 4, (0, 1, 2)), (1025, 6, (1,)), (4097, 4, (0, 2))])
def test_product_columns_alone(ctx, nb, B, reach):
    import torch
    from paper_1002_1202_amd import api
    print(f"case: few columns product nb={nb} B={B}", flush=True)
    pair, _, _ = system(ctx, nb, B, reach)
    rng = np.random.default_rng(nb)
    X = rng.normal(size=(nb * B, 65)) + 1j * rng.normal(size=(nb * B, 65))
    al = rng.uniform(-5, 5, 65) + 0.1j
    Y = api.spmm(ctx, pair, torch.from_numpy(X).cuda(), al).cpu().numpy()
    for R in (1, 2, 8, 9, 63):
        part = torch.from_numpy(np.ascontiguousarray(X[:, :R])).cuda()
        assert np.array_equal(api.spmm(ctx, pair, part, al[:R]).cpu().numpy(), Y[:, :R])


# one and four waves a row (complex64 from 4096 block rows, FP64 from 12288, seed
# product from 4096), short and long rows; column 1 of the two or more is zero and
# never works
@pytest.mark.parametrize("nb,B,R,reach,precision",
                         [(4096, 4, 1, (0, 1), "mixed"), (4096, 4, 8, (0, 2), "mixed"), (4096, 4, 9, (0, 1), "fp64"),
                          (12289, 4, 2, (0, 1), "fp64"), (4095, 6, 8, (0, 1), "mixed"), (512, 6, 8, (9, 10), "fp64"),
                          (300, 6, 130, (9, 10), "mixed")])
def test_solve_few_columns(ctx, nb, B, R, reach, precision):
    from paper_1002_1202_amd import api
    print(f"case: few columns solve nb={nb} B={B} R={R} {precision}", flush=True)
    pair, S, H = system(ctx, nb, B, reach)
    N = nb * B
    rng = np.random.default_rng(R)
    b = rng.normal(size=(R, N)) + 1j * rng.normal(size=(R, N))
    b /= np.linalg.norm(b, axis=1)[:, None]
    if R > 1:
        b[1] = 0
    z = np.array([-3 + 0.5j, 1 + 0.5j])
    res = api.solve(ctx, pair, z, B=b, tol=1e-12, precision=precision)
    assert res.status == 0 and res.converged.all()
    for k, zk in enumerate(z):
        # |x - x_k| <= |A^-1| tol |b|: A's smallest singular value is at least Im z
        # times S's smallest eigenvalue (0.6 by its rows), with a factor of ten
        X = spl.splu((zk * S - H).tocsc()).solve(np.ascontiguousarray(b.T))
        assert np.linalg.norm(res.G_cols[k].T - X, axis=0).max() <= 10 * 1e-12 / (0.5 * 0.6)
        if R > 1:
            assert not res.G_cols[k, 1].any()
