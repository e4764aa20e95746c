"""H-matrix products at the edges of their tiles: 16 pad columns of a leaf (leaves of 9, 18 or 19
columns and one of 150), 8 right-hand sides, 16 terms of a block, four interface columns a step,
against the oracle's dense product.

Tolerance: entries of the table within 1e-13 of the oracle's and FP64 sums of 6 n_i terms, 1e-10 of
the product's norm where nothing is compressed; 1e-9 with a compression bound of 1e-12."""
import numpy as np
import pytest

import fbc_workloads as W
from oracle import green

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,tol", [(dict(b_min=20, max_rank=1), 1e-10), (dict(b_min=10, max_rank=1), 1e-10),
                                    (dict(b_min=200), 1e-10), (dict(b_min=20, eps=1e-12, max_rank=512), 1e-9)])
@pytest.mark.parametrize("R", [1, 8, 11])
def test_product_at_tile_edges(R, kw, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC, HMatrix
    wl = W.make_custom(4, 149, 150, R, 128, seed=R)
    c = wl.cells[0]
    ctx = FBC(wl.cells, wl.bz, form="dtable_fp64")
    h = HMatrix(ctx, **{"gamma": 2, **kw})
    rng = np.random.default_rng(R)
    x = rng.normal(size=(3, 3 * c.n_i, R, 2))
    y = torch.full((3, 3 * c.n_b, R, 2), float("nan"), dtype=torch.float64, device="cuda")
    h.apply(torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    got = y.cpu().numpy() @ np.array([1, 1j])
    g = green.green_modes_dense(c.nz, 128, 128, c.cols_b, c.cols_i)
    for m in range(3):
        ref = g[m] @ (x[m] @ np.array([1, 1j]))
        assert np.linalg.norm(got[m] - ref) < tol * np.linalg.norm(ref), m
    if kw.get("max_rank") == 512:
        assert h.info.max_rank_used > 16
    # inside the update: records of whole groups of 8 right-hand sides
    f = torch.from_numpy(c.forces).cuda()
    w = [torch.full((R, c.nz, c.n_b, 3), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2)]
    ctx.green_apply(f, w[0])
    ctx.set_hmat(h)
    ctx.green_apply(f, w[1])
    assert ctx.sync_status() == 0
    assert torch.linalg.norm(w[1] - w[0]) < tol * torch.linalg.norm(w[0])
    ctx.set_hmat(None)
    h.close()
    ctx.close()
