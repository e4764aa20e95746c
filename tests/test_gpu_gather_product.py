"""Reduced products gathered from the table of column offsets: 128 rows per job (42 2/3 pad
columns), K chunks of 32 complex columns (10 2/3 interface columns), 1, 2 and 4 column tiles, 8
tiles as two jobs, against the FP64 oracle and against the streamed store.

Tolerance, per component, as a multiple of sum |G^||f^| over its row and all modes: FP32 sums over
at most 256 real terms (384 with the three partial products of the split forms over 128), each
rounded once, plus the representation of the operands -- 2^-24 for FP32, 2^-21 for two FP16
halves, 2^-15 for two BF16 halves (the dropped product of the low halves included) -- is below
400 2^-24 and 400 2^-24 + 2^-15."""
import numpy as np
import pytest
import torch

import fbc_workloads as W
from oracle import apply as oap, green as ogr

pytestmark = pytest.mark.gpu

BOUND = {"fp32": 400 * 2.0 ** -24, "split_fp16": 400 * 2.0 ** -24, "split_bf16": 400 * 2.0 ** -24 + 2.0 ** -15}


def _run(cells, bz, form, lists=((1, 2),), **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import FBC
    dev = torch.device("cuda:0")
    ctx = FBC(cells, bz, form=form, row_gauge=False, **kw)
    f = torch.from_numpy(np.concatenate([c.forces.ravel() for c in cells])).to(dev)
    w = torch.full((ctx.info.u_elems,), float("nan"), dtype=torch.float64, device=dev)
    outs = []
    for nsplit, order in lists:
        for v in range(ctx.info.n_variants):
            ctx.set_kernel_variant(v)
            ctx.set_work_list(nsplit, order)
            ctx.green_apply(f, w)
            assert ctx.sync_status() == 0
            outs.append(w.cpu().numpy())
    store = ctx.info.store_bytes
    ctx.close()
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])
    return outs[0], store


def _against_oracle(cells, bz, form, got):
    at = 0
    for c in cells:
        g = ogr.green_modes_dense(c.nz, bz, bz, c.cols_b, c.cols_i)
        ref = oap.apply_green(g, c.forces)
        fh = np.abs(oap.line_rfft(c.forces)).reshape(c.n_rhs, c.nz // 2 + 1, -1)
        scale = sum(2 * fh[:, m] @ np.abs(g[m]).T for m in range(fh.shape[1])) / c.nz     # [R, 3 n_b]
        err = np.abs(got[at:at + ref.size].reshape(ref.shape) - ref).max(axis=1).reshape(c.n_rhs, -1)
        at += ref.size
        assert (err <= BOUND[form] * scale).all(), (c.nz, c.n_i, c.n_b, c.n_rhs, (err / scale).max())


@pytest.mark.parametrize("form", ["fp32", "split_fp16", "split_bf16"])
@pytest.mark.parametrize("n_i,n_b", [(1, 1), (10, 42), (11, 43), (21, 85), (22, 86), (33, 128), (65, 171)])
@pytest.mark.parametrize("R", [1, 9, 17, 40])
def test_tile_edges(n_i, n_b, R, form):
    cells = W.make_custom(4, n_i, n_b, R, 32, seed=100 * n_i + R, zero_net_force=n_i > 1).cells
    kw = {"check_netforce": False} if n_i == 1 else {}
    got, _ = _run(cells, 32, form, ((1, 2), (1, 0), (1, 3), (1, 4)), **kw)
    _against_oracle(cells, 32, form, got)


@pytest.mark.parametrize("form", ["fp32", "split_fp16", "split_bf16"])
@pytest.mark.parametrize("rhs", [(3, 16), (64, 2, 30)])
def test_cells_of_different_tile_counts(rhs, form):
    cells = []
    for k, r in enumerate(rhs):
        cells += W.make_custom(8 >> (k & 1), 20 + 27 * k, 60 + 39 * k, r, 32, seed=k).cells
    got, _ = _run(cells, 32, form)
    _against_oracle(cells, 32, form, got)


@pytest.mark.parametrize("form", ["fp32", "split_fp16", "split_bf16"])
@pytest.mark.parametrize("R", [5, 13, 30, 60])
@pytest.mark.parametrize("nsplit", [1, 3])
def test_gathered_equals_streamed(R, nsplit, form):
    """Pad columns in a random order: their boxes of offsets do not fit, the blocks are stored and
    streamed.  Without skipping every row is then the same sum over the same operands."""
    cell = W.make_custom(8, 130, 430, R, 64, seed=R).cells[0]
    a, sa = _run([cell], 64, form, ((nsplit, 2),), skip_tol=-1.0)
    perm = np.random.default_rng(7).permutation(cell.n_b)
    mixed = W.Cell(cell.nz, cell.cols_i, np.ascontiguousarray(cell.cols_b[perm]), cell.n_rhs, cell.forces)
    b, sb = _run([mixed], 64, form, ((nsplit, 2),), skip_tol=-1.0)
    assert sb > 2 * sa
    shape = (R, cell.nz, cell.n_b, 3)
    assert np.array_equal(a.reshape(shape)[:, :, perm], b.reshape(shape))
