"""Products on a caller's own X and Y: column counts around the chunks of 64 and
the 128 factors of a launch, one factor for all columns, and Y over X."""
import numpy as np
import pytest

from test_gpu_shared_rows import block_product, chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("same", [False, True])
@pytest.mark.parametrize("entry", ["spmm", "spmm in place", "noalloc", "noalloc in place", "host"])
@pytest.mark.parametrize("nb,B,R", [(1, 4, 1), (5, 6, 63), (37, 4, 65), (41, 6, 128), (33, 4, 129), (700, 6, 250),
                                    (4100, 4, 131), (20, 4, 300), (9, 6, 512), (9, 4, 513), (9, 4, 1025)])
def test_product_vs_numpy(nb, B, R, entry, same):
    import torch
    from paper_1002_1202_amd import _lib, api
    print(f"case: product nb={nb} B={B} R={R} {entry} same={same}", flush=True)
    ctx = api.Context(0)
    rng = np.random.default_rng(nb + R)
    reach = (0, 1, 2)
    rowptr, colidx, H, S = chain(rng, nb, B, reach)
    pair = api.Pair(ctx, B, rowptr, colidx, H=H, S=S)
    X = rng.normal(size=(nb * B, R)) + 1j * rng.normal(size=(nb * B, R))
    z = np.full(R, -3.25 + 0.5j) if same else rng.uniform(-20, 5, R) + 0.05j
    Xd = torch.from_numpy(X).cuda()
    if entry.startswith("noalloc") and R % 64 and 32 * nb * B * -(-R // 64) * 64 > 64 << 20:
        # refused, as with the padded copies that its limit stands for
        with pytest.raises(RuntimeError, match="scratch"):
            api.spmm_noalloc(ctx, pair, Xd, z)
        return
    if entry == "host":
        Y = api.spmm(ctx, pair, X, z)
    elif entry == "spmm":
        Y = api.spmm(ctx, pair, Xd, z).cpu().numpy()
    elif entry == "noalloc" or (entry == "noalloc in place" and R % 64 == 0):   # full chunks in place: not offered
        Y = api.spmm_noalloc(ctx, pair, Xd, z).cpu().numpy()
    elif entry == "noalloc in place":
        Y = api.spmm_noalloc(ctx, pair, Xd, z, Y=Xd).cpu().numpy()
    else:
        a = api._complex_view(z.astype(np.complex128))
        _lib.check(ctx.lib.gsc_spmm(ctx.h, pair.h, R, api._ptr(a), api._vp(Xd), api._vp(Xd), _lib.MEM_DEVICE))
        Y = Xd.cpu().numpy()
    SX, SA = block_product(rowptr, colidx, S, X)
    HX, HA = block_product(rowptr, colidx, H, X)
    # rounding of two sums of n terms each, a complex scale and a difference
    n = B * (2 * max(reach) + 1)
    bound = 4 * (n + 4) * np.finfo(float).eps * (np.abs(z) * SA + HA)
    assert np.all(np.abs(Y - (z * SX - HX)) <= bound)
