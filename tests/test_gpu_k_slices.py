"""K slices of the reduced products where row tiles are few: eight where four would leave most of the
chip idle (many interface columns, few pad columns), four or fewer elsewhere, against the oracle.
Tolerance: the forms' bounds elsewhere, 1e-6, and 2e-5 for split BF16."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,tol", [("fp32", 1e-6), ("split_fp16", 1e-6), ("split_bf16", 2e-5)])
@pytest.mark.parametrize("n_i,n_b,R,slices", [(350, 40, 1, 8), (347, 30, 20, 8), (330, 40, 1, 4), (60, 300, 3, 1)])
def test_slices(n_i, n_b, R, slices, form, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    c = W.make_custom(16, n_i, n_b, R, 128, seed=n_i).cells[0]
    ctx = FBC([c], 128, form=form)
    assert ctx.info.nsplit == slices
    w = torch.full((R, 16, n_b, 3), float("nan"), dtype=torch.float64, device="cuda")
    ctx.green_apply(torch.from_numpy(c.forces).cuda(), w)
    assert ctx.sync_status() == 0
    ctx.close()
    ref = oap.apply_green(ogr.green_modes_dense(16, 128, 128, c.cols_b, c.cols_i), c.forces)
    assert np.linalg.norm(w.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
