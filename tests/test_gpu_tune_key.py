"""The autotune cache keeps contexts apart that differ in the precision of the table product only: its
FP32 jobs are another kernel, and a choice timed for one is none for the other."""
import pytest
import torch

import fbc_workloads as W

pytestmark = pytest.mark.gpu


def test_table_fp32_has_a_key_of_its_own(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    c = W.make_custom(32, 60, 100, 9, 32, seed=4).cells[0]
    path = str(tmp_path / "tune.txt")
    f = torch.from_numpy(c.forces).cuda()
    w = torch.zeros((c.n_rhs, c.nz, c.n_b, 3), dtype=torch.float64, device="cuda")
    for k, fp32 in enumerate((False, True, False, True)):
        ctx = FBC([c], 32, form="dtable_fp64", table_fp32=fp32)
        assert ctx.autotune(f, w, reps=1, cache=path)["from_cache"] == (k >= 2)
        ctx.close()
    assert len(open(path).read().splitlines()) == 2
