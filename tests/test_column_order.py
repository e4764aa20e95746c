"""Columns that the caller lists in no neighbourly order.  The offset-table products take them by angle
(plan_order: tests/order_check.cpp under the sanitizers); on the GPU every route through that order --
product, response, relaxation, H-matrix, learned form, block rows -- against the oracle or against the same
cell with its columns by angle.

Tolerance: FP64 sums of at most 6 n_i terms in another order, 1e-10 against the oracle (the bound
elsewhere) and 1e-12 between two orders; with table_fp32 1e-6."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr
from test_plan_sanitized import CSRC, HERE

ORDERS = {
    "random": lambda c, seed: np.random.default_rng(seed).permutation(len(c)),
    "distance": lambda c, seed: np.argsort(c[:, 0] ** 2 * 3 + 4 * c[:, 0] * c[:, 1] + 4 * c[:, 1] ** 2, kind="stable"),
    "index": lambda c, seed: np.lexsort((c[:, 1], c[:, 0])),
    "angle": lambda c, seed: np.arange(len(c)),
}


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_order_under_sanitizers(tmp_path):
    exe = str(tmp_path / "order_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I",
                    CSRC, os.path.join(CSRC, "plan.cpp"), os.path.join(HERE, "order_check.cpp"), "-o", exe], check=True,
                   capture_output=True, timeout=300)
    geo = str(tmp_path / "geometry.bin")
    sets = [(s, oi, ob) for s in ((1, 1), (1, 70000), (96, 192), (300, 600)) for oi, ob in
            (("angle", "angle"), ("index", "index"), ("random", "angle"), ("angle", "distance"), ("random", "random"))]
    with open(geo, "wb") as fp:
        np.asarray([len(sets)], dtype=np.int32).tofile(fp)
        for (n_i, n_b), oi, ob in sets:
            if n_b == 70000:                 # one interface column, pad columns in a row
                ci, cb = np.zeros((1, 2), np.int32), np.stack([np.arange(1, 70001), np.zeros(70000)], 1).astype(np.int32)
                oi = ob = "angle"
            else:
                ci, cb = W.ring_columns(n_i, n_b)
            far = ("random", "distance")
            want = (oi in far) + 2 * (ob in far) if n_i * n_b >= 65536 else 0
            ci, cb = ci[ORDERS[oi](ci, 1)], cb[ORDERS[ob](cb, 2)]
            np.asarray([1, len(ci), len(cb)], dtype=np.int32).tofile(fp)
            np.ascontiguousarray(ci, dtype=np.int32).tofile(fp)
            np.ascontiguousarray(cb, dtype=np.int32).tofile(fp)
            np.asarray([want], dtype=np.int32).tofile(fp)
    r = subprocess.run([exe, geo], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def _cells(nz, n_i, n_b, R, orders, bz=128):
    """The cell by angle, and the same with its columns in other orders."""
    c = W.make_custom(nz, n_i, n_b, R, bz, seed=n_b).cells[0]
    pi, pb = ORDERS[orders[0]](c.cols_i, 3), ORDERS[orders[1]](c.cols_b, 4)
    m = W.Cell(nz, np.ascontiguousarray(c.cols_i[pi]), np.ascontiguousarray(c.cols_b[pb]), R,
               np.ascontiguousarray(c.forces[:, :, pi]))
    return c, m, pb


def _response(cell, **kw):
    from paper_2105_08798_amd import FBC
    ctx = FBC([cell], 128, **kw)
    w = torch.full((cell.n_rhs, cell.nz, cell.n_b, 3), float("nan"), dtype=torch.float64, device="cuda")
    ctx.green_apply(torch.from_numpy(cell.forces).cuda(), w)
    assert ctx.sync_status() == 0
    return ctx, w.cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("orders", [("random", "random"), ("angle", "random"), ("distance", "angle"), ("index", "index")])
@pytest.mark.parametrize("form,kw,tol", [("fp64", {}, 1e-10), ("dtable_fp64", {"table_fp32": True}, 1e-6),
                                         ("fp32", {}, 1e-6), ("split_fp16", {}, 1e-6)])
@pytest.mark.parametrize("nz,n_i,n_b,R", [(8, 181, 401, 3), (64, 200, 333, 9)])
def test_products(nz, n_i, n_b, R, form, kw, tol, orders):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _, cell, _ = _cells(nz, n_i, n_b, R, orders)
    ctx, w = _response(cell, form=form, **kw)
    ref = oap.apply_green(ogr.green_modes_dense(nz, 128, 128, cell.cols_b, cell.cols_i), cell.forces)
    assert np.linalg.norm(w - ref) <= tol * np.linalg.norm(ref)
    if form == "fp64":
        # the blocks that fbc_copy_block_rows gives (windows included) are the product's
        fh, wh = np.fft.rfft(cell.forces, axis=1), np.fft.rfft(w, axis=1)
        for m in (0, nz // 4, nz // 2):
            a = ctx.block_rows(0, m, 7, n_b - 3, n_i)
            got = np.einsum("kj,rj->rk", a, fh[:, m].reshape(R, -1))
            assert np.linalg.norm(got - wh[:, m, 7:n_b - 3].reshape(R, -1)) <= 1e-12 * np.linalg.norm(wh[:, m])
    ctx.close()


@pytest.mark.gpu
def test_update_and_relaxation():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    base, cell, pb = _cells(32, 200, 340, 4, ("random", "distance"))
    other = W.make_custom(16, 60, 100, 2, 128, seed=3).cells[0]           # a cell beside it that keeps its order
    out = []
    for c in (base, cell):
        ctx = FBC([other, c], 128, form="fp64")
        f = torch.from_numpy(np.concatenate([other.forces.ravel(), c.forces.ravel()])).cuda()
        u0 = np.random.default_rng(5).normal(size=(4, 32, 340, 3))
        v = np.random.default_rng(6).normal(size=other.n_rhs * 16 * 100 * 3)
        u = torch.from_numpy(np.concatenate([v, (u0 if c is base else u0[:, :, pb]).ravel()])).cuda()
        ctx.apply(f, u, alpha=0.7)
        ctx.relax_begin(relax=True, du_max=0.05, tol_f=1e-3)
        for _ in range(3):
            ctx.relax_step(f, u)
        assert ctx.sync_status() == 0
        ctx.close()
        a = u.cpu().numpy()
        out.append((a[:v.size], a[v.size:].reshape(4, 32, 340, 3)))
    assert np.abs(out[0][0] - out[1][0]).max() <= 1e-12 * np.abs(out[0][0]).max()
    assert np.abs(out[0][1][:, :, pb] - out[1][1]).max() <= 1e-12 * np.abs(out[0][1]).max()


@pytest.mark.gpu
def test_hmatrix_and_learned_form():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC, MLP, HMatrix, Surrogate
    base, cell, pb = _cells(16, 200, 340, 3, ("random", "random"))
    f = torch.from_numpy(cell.forces).cuda()
    ctx, w = _response(cell, form="dtable_fp64")
    h = HMatrix(ctx, eps=1e-10, max_rank=16)
    ctx.set_hmat(h)
    y = torch.full((3, 16, 340, 3), float("nan"), dtype=torch.float64, device="cuda")
    ctx.green_apply(f, y)
    assert ctx.sync_status() == 0
    ctx.set_hmat(None)
    h.close()
    ctx.close()
    assert np.abs(y.cpu().numpy() - w).max() <= 1e-7 * np.abs(w).max()
    net = MLP(64, seed=1)
    sur = Surrogate(r_c=6.0)
    sur.set_mlp(net)
    got = []
    for c in (base, cell):
        ctx, w = _response(c, form="surrogate", surrogate=sur)
        ctx.close()
        got.append(w)
    assert np.abs(got[0][:, :, pb] - got[1]).max() <= 1e-12 * np.abs(got[0]).max()
    sur.close()
    net.close()
