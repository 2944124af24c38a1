"""Small systems, one workgroup per column: workgroup sizes at their edges, rows
longer than the blocks kept in registers, columns beyond the CUs, seed switches
and restarts, a cut iteration, and the tiled kernels on the same inputs."""
import numpy as np
import pytest

from oracle import green as ogreen
from test_gpu_shared_rows import chain

pytestmark = pytest.mark.gpu

Z = np.array([-3 + 3j, -4 + 0.3j, -1 + 0.3j, 0.5 + 0.4j, 2 + 0.3j])


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_1002_1202_amd import api
    assert torch.cuda.is_available()
    return api.Context(0)


def system(ctx, nb, B, reach):
    from paper_1002_1202_amd import api
    rowptr, colidx, H, S = chain(np.random.default_rng(nb * B), nb, B, reach)
    row = np.repeat(np.arange(nb), np.diff(rowptr))
    Sd, Hd = np.zeros((nb, B, nb, B)), np.zeros((nb, B, nb, B))
    Sd[row, :, colidx, :], Hd[row, :, colidx, :] = S, H
    N = nb * B
    return api.Pair(ctx, B, rowptr, colidx, H=H, S=S), Hd.reshape(N, N), Sd.reshape(N, N), row, colidx


# 256, 512, 768 and 1024 threads (N = 128, 256, 384, 512) and one block row
# more; rows of one block and beyond 4 x 7; more columns than CUs (264)
SIZES = [(1, 4, 2, (0,)), (3, 4, 12, (0, 1)), (32, 4, 70, (0, 1, 15)), (33, 4, 7, (1, 2)), (64, 4, 256, (0, 3)),
         (65, 4, 264, (15,)), (96, 4, 65, (1, 2)), (97, 4, 5, (10,)), (128, 4, 64, (0, 1, 15)), (129, 4, 3, (1,)),
         (1, 6, 1, (0,)), (21, 6, 126, (0, 1, 15)), (22, 6, 5, (1, 2)), (42, 6, 64, (2, 16)), (43, 6, 9, (0, 1)),
         (64, 6, 264, (0, 9)), (65, 6, 66, (15,)), (85, 6, 64, (1, 2)), (86, 6, 2, (1,))]


@pytest.mark.parametrize("carry", ["full", "projected"])
@pytest.mark.parametrize("nb,B,R,reach", SIZES)
def test_solve_vs_dense(ctx, nb, B, R, reach, carry):
    from paper_1002_1202_amd import api
    print(f"case: small nb={nb} B={B} R={R} reach={reach} {carry}", flush=True)
    pair, H, S, _, _ = system(ctx, nb, B, reach)
    N = nb * B
    rng = np.random.default_rng(R)
    rhs = rng.integers(0, N, R)
    proj = np.stack([rhs, rng.integers(0, N, R), rng.integers(0, N, R)], 1)
    # the seed is the shift that converges first, so the others outlive it
    res = api.solve(ctx, pair, Z, rhs=rhs, tol=1e-12, carry=carry, proj=proj, seed_index=0,
                    precision="mixed" if nb % 2 else "fp64")
    assert res.status == 0 and res.converged.all()
    if nb > 20:
        assert (res.switches if carry == "full" else res.restarts) > 0
    X = ogreen.solve_dense(H, S, Z, rhs)
    # |x - x_k| <= |A^-1| tol: A's smallest singular value is at least Im z times
    # S's smallest eigenvalue (0.6 by its rows), with a factor of ten
    bound = 10 * 1e-12 / (0.3 * 0.6)
    ref = np.take_along_axis(X, np.broadcast_to(proj[None], (len(Z),) + proj.shape), axis=2)
    assert np.abs(res.G_proj - ref).max() <= bound
    if carry == "full":
        assert np.linalg.norm(res.G_cols - X, axis=2).max() <= bound


@pytest.mark.parametrize("nb,B,reach", [(1, 4, (0,)), (32, 4, (0, 15)), (50, 4, (1, 2)), (21, 6, (0, 1, 15)),
                                        (60, 6, (1,))])
def test_band_gradient_vs_dense(ctx, nb, B, reach):
    from paper_1002_1202_amd import api
    print(f"case: small gradient nb={nb} B={B} reach={reach}", flush=True)
    pair, H, S, row, col = system(ctx, nb, B, reach)
    w = np.array([0.2, 0.5, -0.3, 0.8, 0.4])
    dH, dS, E, _ = api.band_energy_vjp(ctx, pair, Z, w, tol=1e-13, seed_index=0)
    gH, gS = ogreen.band_energy_grad_dense(H, S, Z, w)
    for a, g in ((dH, gH), (dS, gS)):
        g = g.reshape(nb, B, nb, B)[row, :, col, :]
        # a product of two Green's functions, each within 10 tol / 0.18 as above
        assert np.abs(a - g).max() <= 1e-9 * np.abs(g).max()


@pytest.mark.parametrize("carry", ["full", "projected"])
@pytest.mark.parametrize("max_iter", [1, 4, 17, 400])
def test_same_as_tiles(ctx, max_iter, carry):
    """Dense right-hand sides, one of them zero, stopped after max_iter
    iterations: the tiled kernels (which per-kernel timing selects) see the
    same recurrences."""
    from paper_1002_1202_amd import api
    print(f"case: small as tiles max_iter={max_iter} {carry}", flush=True)
    pair, _, _, _, _ = system(ctx, 40, 4, (0, 1, 2))
    rng = np.random.default_rng(3)
    b = rng.normal(size=(9, 160)) + 1j * rng.normal(size=(9, 160))
    b[4] = 0
    proj = rng.integers(0, 160, (9, 2))
    out = []
    for on in (False, True):
        api.profile_enable(ctx, on)
        try:
            out.append(api.solve(ctx, pair, Z, B=b, tol=1e-11, max_iter=max_iter, carry=carry, proj=proj,
                                 seed_index=0, fuse_steps=5))
        finally:
            api.profile_enable(ctx, False)
    s, t = out
    assert s.status == t.status and np.array_equal(s.converged, t.converged)
    if max_iter < 400:
        # equal recurrences: rounding (and the inner solve's 1e-13) grown over
        # at most 17 steps
        assert s.shift_rhs_iters == t.shift_rhs_iters and s.outer_iters == t.outer_iters
        tol = 1e-9
        assert np.abs(s.res - t.res).max() <= tol * np.abs(t.res).max()
    else:
        tol = 2 * 10 * 1e-11 / (0.3 * 0.6)   # both within tol |A^-1| of the solution
    nb_ = np.linalg.norm(b, axis=1).max()
    assert np.abs(s.G_proj - t.G_proj).max() <= tol * nb_ / 0.18
    if carry == "full":
        assert np.abs(s.G_cols - t.G_cols).max() <= tol * nb_ / 0.18
        assert not s.G_cols[:, 4].any()
