"""Lines of 4096 layers, the longest that a cell may have: the update and the relaxation step, with
and without the force checks, for forces with net force per layer (the reduced forms then transform
it along the line, one component at a time at this length), against the oracle.

Tolerance: the forms' own elsewhere, 1e-10 for FP64 and 1e-6 for split FP16 (blocks and forces held
to 2^-22; the transforms are FP64 and add 12 roundings of 2^-53)."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("du_max", [0.0, 1e6])
@pytest.mark.parametrize("check,project", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("form,tol", [("fp64", 1e-10), ("split_fp16", 1e-6)])
def test_4096_layers(form, tol, check, project, du_max):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC, RELAX_OUT_DOUBLES, parse_relax_out
    nz, n_i, n_b, R = 4096, 5, 9, 3
    c = W.make_custom(nz, n_i, n_b, R, 16, seed=41, zero_net_force=False).cells[0]
    force = c.forces - c.forces.mean(axis=(1, 2), keepdims=True)
    assert np.abs(force.sum(axis=2)).max() > 1e-2
    ctx = FBC([c], 16, form=form, check_netforce=check, project_netforce=project)
    f = torch.from_numpy(force).cuda()
    u0 = np.random.default_rng(2).normal(size=(R, nz, n_b, 3)) * 0.01
    u = torch.from_numpy(u0.copy()).cuda()
    ctx.apply(f, u, alpha=0.7)
    assert ctx.sync_status() == 0
    v = torch.from_numpy(u0.copy()).cuda()
    ctx.relax_begin(relax=True, du_max=du_max, tol_f=1e-3)
    out = torch.zeros(R * RELAX_OUT_DOUBLES, dtype=torch.float64, device="cuda")
    ctx.relax_step(f, v, out)
    assert ctx.sync_status() == 0
    ctx.close()
    w = oap.apply_green(ogr.green_modes_dense(nz, 16, 16, c.cols_b, c.cols_i), force)
    for got, alpha in ((u, 0.7), (v, 1.0)):
        want = oap.pad_update(u0, w, alpha)[0]
        assert np.abs(got.cpu().numpy() - want).max() <= tol * np.abs(w).max() + 1e-14 * np.abs(u0).max()
    for r, o in enumerate(parse_relax_out(out)):
        assert o["alpha"] == 1.0 and abs(o["f_inf"] - np.abs(force[r]).max()) <= 1e-15 * o["f_inf"]
        assert abs(o["step_inf"] - np.abs(w[r]).max()) <= tol * np.abs(w).max()
