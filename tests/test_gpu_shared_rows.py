"""Block rows shared by the waves of a workgroup: rows of fewer stored blocks
than waves, row groups that take several rows, both splits of the two-matrix
products, and launches beyond the grid's second dimension."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1002_1202_amd import api
    assert torch.cuda.is_available()
    return api.Context(0)


def chain(rng, nb, B, reach):
    """Blocks |I - J| <= reach[min(I, J)] of a chain: rows of 1 to 2 max(reach) + 1
    blocks; S diagonally dominant, H symmetric."""
    r = np.asarray(reach)[rng.integers(0, len(reach), nb)]
    pairs = [(i, i + d) for i in range(nb) for d in range(1, r[i] + 1) if i + d < nb]
    i, j = (np.array(v, np.int64) for v in zip(*pairs)) if pairs else (np.zeros(0, np.int64),) * 2
    rows, cols = np.concatenate([i, j, np.arange(nb)]), np.concatenate([j, i, np.arange(nb)])
    Sp, Hp = (rng.uniform(-1, 1, (len(i), B, B)) for _ in range(2))
    d = rng.uniform(-1, 1, (nb, B, B))
    S = np.concatenate([Sp, Sp.transpose(0, 2, 1), np.zeros((nb, B, B))]) * (0.4 / (B * (2 * max(reach) + 1)))
    S[len(rows) - nb:] = np.eye(B)
    H = np.concatenate([Hp, Hp.transpose(0, 2, 1), d + d.transpose(0, 2, 1)])
    order = np.argsort(rows * nb + cols)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=nb))]).astype(np.int64)
    return rowptr, cols[order].astype(np.int32), H[order], S[order]


def block_product(rowptr, colidx, M, X):
    """M X and |M| |X| for one real block matrix, in numpy."""
    B = M.shape[1]
    Xb = X.reshape(-1, B, X.shape[1])
    Y, A = np.zeros_like(Xb), np.zeros(Xb.shape)
    for k in range(int(np.diff(rowptr).max())):
        b = rowptr[:-1] + k
        row = np.flatnonzero(b < rowptr[1:])
        b = b[row]
        for c in range(B):
            Y[row] += M[b][:, :, c, None] * Xb[colidx[b]][:, None, c]
            A[row] += np.abs(M[b][:, :, c, None]) * np.abs(Xb[colidx[b]][:, None, c])
    return Y.reshape(X.shape), A.reshape(X.shape)


# nb * chunks below, at and beyond 8192 (the two-matrix split), nb beyond one
# grid dimension, ragged columns
@pytest.mark.parametrize("nb,B,R,reach", [(5, 4, 3, (0,)), (63, 6, 64, (0, 1)), (130, 4, 129, (0, 1, 2)),
                                          (4095, 4, 128, (0, 1, 2)), (4096, 4, 128, (0, 1, 3)),
                                          (2731, 6, 190, (1, 2)), (65537, 4, 2, (0, 1))])
def test_product_vs_numpy(ctx, nb, B, R, reach):
    import torch
    from paper_1002_1202_amd import api
    print(f"case: product nb={nb} B={B} R={R} reach={reach}", flush=True)
    rng = np.random.default_rng(nb + R)
    rowptr, colidx, H, S = chain(rng, nb, B, reach)
    pair = api.Pair(ctx, B, rowptr, colidx, H=H, S=S)
    X = rng.normal(size=(nb * B, R)) + 1j * rng.normal(size=(nb * B, R))
    z = rng.uniform(-20, 5, R) + 0.05j
    Y = api.spmm(ctx, pair, torch.from_numpy(X).cuda(), z).cpu().numpy()
    SX, SA = block_product(rowptr, colidx, S, X)
    HX, HA = block_product(rowptr, colidx, H, X)
    # rounding of two sums of n terms each, a complex scale and a difference
    n = B * (2 * max(reach) + 1)
    bound = 4 * (n + 4) * np.finfo(float).eps * (np.abs(z) * SA + HA)
    assert np.all(np.abs(Y - (z * SX - HX)) <= bound)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nb,B,R,reach", [(40, 4, 70, (0,)), (30, 6, 9, (0, 1)), (1100, 4, 3, (0, 1, 2))])
def test_solve_vs_dense(ctx, nb, B, R, reach, precision):
    from paper_1002_1202_amd import api
    print(f"case: solve nb={nb} B={B} R={R} reach={reach} {precision}", flush=True)
    rng = np.random.default_rng(nb)
    rowptr, colidx, H, S = chain(rng, nb, B, reach)
    pair = api.Pair(ctx, B, rowptr, colidx, H=H, S=S)
    N = nb * B
    rhs = np.sort(rng.choice(N, size=R, replace=False)).astype(np.int64)
    z = np.linspace(-4, 4, 5) + 0.3j
    res = api.solve(ctx, pair, z, rhs=rhs, tol=1e-12, precision=precision)
    row = np.repeat(np.arange(nb), np.diff(rowptr))
    Sd, Hd = np.zeros((nb, B, nb, B)), np.zeros((nb, B, nb, B))
    Sd[row, :, colidx, :], Hd[row, :, colidx, :] = S, H
    Sd, Hd = Sd.reshape(N, N), Hd.reshape(N, N)
    assert res.converged.all()
    E = np.zeros((N, R))
    E[rhs, np.arange(R)] = 1.0
    for k, zk in enumerate(z):
        # |x - x_k| <= |A^-1| tol: A's smallest singular value is at least Im z
        # times S's smallest eigenvalue (0.6 by its rows), with a factor of ten
        X = np.linalg.solve(zk * Sd - Hd, E)
        err = np.linalg.norm(res.G_cols[k].T - X, axis=0)
        assert err.max() <= 10 * 1e-12 / (0.3 * 0.6)
