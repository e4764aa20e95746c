"""FP32 products with more than 56 right-hand sides: one job of eight column tiles per row tile
(contexts with a cell of 48 or fewer beside them, or with fewer than 256 row tiles, keep jobs of
four), against the oracle, and both kernel variants bitwise alike.  Tolerance: the form's bound
elsewhere, 1e-6."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("balanced", [True, False])
@pytest.mark.parametrize("tiles,cells", [(8, [(512, 12, 21, 57)]), (8, [(64, 130, 341, 64)]), (4, [(64, 30, 298, 64)]),
                                         (8, [(16, 40, 43, 64), (512, 25, 90, 49)]),
                                         (4, [(16, 40, 43, 64), (512, 25, 90, 48)]), (4, [(512, 12, 21, 56)])])
def test_wide_jobs(tiles, cells, balanced):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    cs = [W.make_custom(nz, n_i, n_b, R, 64, seed=n_b + R, zero_net_force=False).cells[0] for nz, n_i, n_b, R in cells]
    for c in cs:
        c.forces = c.forces - c.forces.mean(axis=2 if balanced else (1, 2), keepdims=True)
    ctx = FBC(cs, 64, form="fp32")
    assert f"CT={tiles} " in ctx.info.kernel_shape.decode()
    f = torch.from_numpy(np.concatenate([c.forces.ravel() for c in cs])).cuda()
    n = sum(c.n_rhs * c.nz * c.n_b * 3 for c in cs)
    got = []
    for v in (0, 1):
        ctx.set_kernel_variant(v)
        w = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
        ctx.green_apply(f, w)
        assert ctx.sync_status() == 0
        got.append(w.cpu().numpy())
    ctx.close()
    assert (got[0] == got[1]).all()
    at = 0
    for c in cs:
        ref = oap.apply_green(ogr.green_modes_dense(c.nz, 64, 64, c.cols_b, c.cols_i), c.forces)
        w = got[0][at:at + ref.size].reshape(ref.shape)
        at += ref.size
        for r in range(c.n_rhs):
            if np.abs(ref[r]).max() > 1e-12 * np.abs(ref).max():
                assert np.linalg.norm(w[r] - ref[r]) <= 1e-6 * np.linalg.norm(ref[r]), r
