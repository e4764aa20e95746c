"""Products over the offset table at the edges of their tiles: 16 pad columns per job, chunks of
16 interface columns, 8 right-hand sides per column tile, cells of different tile counts in
one context, against the FP64 oracle.

Tolerance: FP64 sums of 6 n_i <= 300 terms, each entry within 1e-13 of the oracle's, so 1e-11
of the largest displacement bounds every component."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu


def _check(cells, bz, form, tol, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    dev = torch.device("cuda:0")
    ctx = FBC(cells, bz, form=form, **kw)
    f = torch.from_numpy(np.concatenate([c.forces.ravel() for c in cells])).to(dev)
    w = torch.full((ctx.info.u_elems,), float("nan"), dtype=torch.float64, device=dev)
    outs = []
    for nsplit, order in ((1, 1), (1, 3), (1, 0), (1, 4)):
        ctx.set_work_list(nsplit, order)
        ctx.green_apply(f, w)
        assert ctx.sync_status() == 0
        outs.append(w.cpu().numpy())
    ctx.close()
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])
    at = 0
    for c in cells:
        g = ogr.green_modes_dense(c.nz, bz, bz, c.cols_b, c.cols_i)
        ref = oap.apply_green(g, c.forces)
        got = outs[0][at:at + ref.size].reshape(ref.shape)
        at += ref.size
        assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (c.nz, c.n_i, c.n_b, c.n_rhs)


@pytest.mark.parametrize("n_i,n_b", [(2, 1), (15, 17), (16, 16), (17, 15), (33, 47), (48, 50)])
@pytest.mark.parametrize("R", [1, 8, 9, 17, 64])
def test_tile_edges(n_i, n_b, R):
    _check(W.make_custom(4, n_i, n_b, R, 32, seed=100 * n_i + R).cells, 32, "dtable_fp64", 1e-11)


@pytest.mark.parametrize("rhs", [(3, 16), (40, 2, 9, 20), (64, 1, 30)])
def test_cells_of_different_tile_counts(rhs):
    cells = []
    for k, r in enumerate(rhs):
        cells += W.make_custom(8 >> (k & 1), 20 + 7 * k, 30 + 9 * k, r, 32, seed=k).cells
    _check(cells, 32, "dtable_fp64", 1e-11)
