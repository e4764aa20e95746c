"""Offset-table products of few row tiles, whose column tiles are shared out over several jobs: against
the oracle, and bitwise the same through every work list and variant (shared out or not, a column
tile is the same sum).  Tolerance: FP64 sums of at most 6 n_i terms, 1e-10; with table_fp32 1e-6."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,kw,tol", [("fp64", {}, 1e-10), ("dtable_fp64", {"table_fp32": True}, 1e-6)])
@pytest.mark.parametrize("cells", [[(8, 20, 40, 64)], [(4, 30, 60, 9)], [(4, 33, 17, 40)], [(8, 17, 40, 57), (4, 16, 20, 3)],
                                   [(64, 40, 100, 24)]])
def test_shared_column_tiles(cells, form, kw, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    cs = [W.make_custom(nz, n_i, n_b, R, 64, seed=n_b + R).cells[0] for nz, n_i, n_b, R in cells]
    f = torch.from_numpy(np.concatenate([c.forces.ravel() for c in cs])).cuda()
    ctx = FBC(cs, 64, form=form, **kw)
    got = []
    for v in range(ctx.info.n_variants):
        ctx.set_kernel_variant(v)
        for order in range(5):
            ctx.set_work_list(1, order)
            w = torch.full((ctx.info.u_elems,), float("nan"), dtype=torch.float64, device="cuda")
            ctx.green_apply(f, w)
            assert ctx.sync_status() == 0
            got.append(w.cpu().numpy())
    ctx.close()
    assert all(np.array_equal(g, got[0]) for g in got)
    at = 0
    for c in cs:
        ref = oap.apply_green(ogr.green_modes_dense(c.nz, 64, 64, c.cols_b, c.cols_i), c.forces)
        w = got[0][at:at + ref.size].reshape(ref.shape)
        at += ref.size
        for r in range(c.n_rhs):
            assert np.linalg.norm(w[r] - ref[r]) <= tol * np.linalg.norm(ref[r]), r
