"""Columns far from the lattice origin, whose keys in the offset lookup need more than 32 bits: the
keys on the CPU (tests/key_check.cpp, undefined-behaviour sanitizer), and on the GPU every form and the
H-matrix, bitwise as for the same columns at the origin (only differences of columns enter)."""
import os
import shutil
import subprocess
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import fbc_workloads as W
from test_plan_sanitized import CSRC, HERE, _write_sets


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_keys_under_sanitizer(tmp_path):
    exe = str(tmp_path / "key_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    os.path.join(CSRC, "plan.cpp"), os.path.join(HERE, "key_check.cpp"), "-o", exe], check=True,
                   capture_output=True, timeout=300)
    geo = str(tmp_path / "geometry.bin")
    _write_sets(geo, [[W.ring_columns(n_i, n_b)] for n_i, n_b in ((1, 1), (96, 192))] +
                [[W.ring_columns(n_i, n_b) for n_i, n_b in ((40, 80), (13, 30))]])
    r = subprocess.run([exe, geo], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["fp64", "dtable_fp64", "fp32", "split_fp16", "hmat"])
def test_far_columns(form):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC, HMatrix
    c = W.make_custom(32, 60, 110, 3, 64, seed=5).cells[0]
    u0 = torch.from_numpy(np.random.default_rng(1).normal(size=(3, 32, 110, 3))).cuda()
    got = []
    for at in ((0, 0), (300000000, -400000000)):
        cell = SimpleNamespace(nz=32, n_i=60, n_b=110, n_rhs=3, cols_i=c.cols_i + np.int32(at),
                               cols_b=c.cols_b + np.int32(at))
        ctx = FBC([cell], 64, form="dtable_fp64" if form == "hmat" else form)
        h = None
        if form == "hmat":
            h = HMatrix(ctx, max_rank=2)          # a bound that most blocks pass: read from the table
            ctx.set_hmat(h)
        u = u0.clone()
        ctx.apply(torch.from_numpy(c.forces).cuda(), u, alpha=0.7)
        assert ctx.sync_status() == 0
        got.append(u.cpu().numpy())
        if h is not None:
            ctx.set_hmat(None)
            h.close()
        ctx.close()
    assert np.isfinite(got[0]).all() and (got[0] == got[1]).all()
