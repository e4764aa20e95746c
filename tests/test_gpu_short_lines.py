"""Updates with few layers (the fused inverse transform from 4 layers on, 64 rows per group at 4 and
8, 32 at 16, 16 at 32), and the removed mean at the edges of its partitions (blocks of 2048 values
up to 32 of them, of 8192 beyond; 32 or fewer partial sums added up by the update itself, more by a
kernel of their own), against the oracle.

Tolerance: FP64 throughout, sums of 6 n_i and, for the mean, of at most 3e5 terms: 1e-10 of the
largest displacement; 2e-5 for split BF16 (16 bits of mantissa, its bound elsewhere too)."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu


def _check(nz, n_i, n_b, R, bz, form, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    c = W.make_custom(nz, n_i, n_b, R, bz, seed=nz + n_b + R).cells[0]
    ctx = FBC([c], bz, form=form)
    f = torch.from_numpy(c.forces).cuda()
    u0 = np.random.default_rng(n_b).normal(size=(R, nz, n_b, 3))
    w = torch.full((R, nz, n_b, 3), float("nan"), dtype=torch.float64, device="cuda")
    ctx.green_apply(f, w)
    u = torch.from_numpy(u0.copy()).cuda()
    ctx.apply(f, u, alpha=0.7)
    # the relaxation step's route: a step factor per RHS on the device (1 in the first step)
    v = torch.from_numpy(u0.copy()).cuda()
    ctx.relax_begin(relax=False, du_max=0.0, tol_f=1e-3)
    out = torch.zeros(R * 8, dtype=torch.float64, device="cuda")
    ctx.relax_step(f, v, out)
    assert ctx.sync_status() == 0
    ctx.close()
    g = ogr.green_modes_dense(nz, bz, bz, c.cols_b, c.cols_i)
    ref = oap.apply_green(g, c.forces)
    assert np.abs(w.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    for got, alpha in ((u, 0.7), (v, 1.0)):
        want = oap.pad_update(u0, ref, alpha)[0]
        assert np.abs(got.cpu().numpy() - want).max() <= tol * np.abs(ref).max() + 1e-14 * np.abs(u0).max() * np.sqrt(u0.size), alpha


@pytest.mark.parametrize("form,tol", [("dtable_fp64", 1e-10), ("split_bf16", 2e-5)])
@pytest.mark.parametrize("nz", [2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("n_b,R", [(1, 1), (21, 2), (22, 3), (43, 9)])
def test_short_lines(nz, n_b, R, form, tol):
    _check(nz, 12, n_b, R, 32, form, tol)


@pytest.mark.parametrize("nz,n_b", [(64, 341), (64, 342), (64, 1365), (64, 1366), (2, 400)])
def test_mean_partitions(nz, n_b):
    _check(nz, 12, n_b, 3, 128, "dtable_fp64", 1e-10)
