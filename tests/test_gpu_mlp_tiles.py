"""MLP loss, gradient and forward pass at the edges of their tiles: work groups of 32 samples,
gradient chunks of 32 samples or more (a multiple of 4, at most 23 chunks), against the FP64 oracle.

Tolerance: forward and backward are chains of FP32 sums of at most 129 terms over four layers each
way, O(1) weights and slopes: a few times 2^-24 sqrt(129) per layer, below 1e-5 of the output and
of each layer's gradient (measured against their 2-norms)."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def _net(n, seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_08798_amd import MLP
    rng = np.random.default_rng(seed)
    net = MLP(max_batch=max(n, 4), seed=3)
    p = (omlp.init_params(rng) + 0.05 * rng.normal(size=omlp.n_params())).astype(np.float32)
    net.params(p)
    x = rng.uniform(-1, 1, size=(n, 8)).astype(np.float32)
    t = rng.normal(size=(n, 12)).astype(np.float32)
    return net, p.astype(np.float64), x, t


@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 31, 32, 33, 65, 1023, 1025, 1029, 2055, 4099])
def test_loss_and_gradient_at_tile_edges(n):
    net, p, x, t = _net(n, n)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y = torch.full((n, 12), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    net.forward(xd, y)
    net.loss_grad(xd, td, loss)
    torch.cuda.synchronize()
    y_ref, _ = omlp.forward(p, x.astype(np.float64))
    l_ref, g_ref = omlp.loss_grad(p, x.astype(np.float64), t.astype(np.float64))
    g = net.grad()
    net.close()
    assert np.linalg.norm(y.cpu().numpy() - y_ref) < 1e-5 * np.linalg.norm(y_ref)
    assert abs(loss.item() - l_ref) < 1e-5 * l_ref
    off = 0
    for i, o in zip(omlp.SIZES[:-1], omlp.SIZES[1:]):
        for sl in (slice(off, off + o * i), slice(off + o * i, off + o * i + o)):
            assert np.linalg.norm(g[sl] - g_ref[sl]) < 1e-5 * np.linalg.norm(g_ref[sl]), (i, o)
        off += o * i + o


@pytest.mark.parametrize("shift", [0, 3, 8 * 40])
def test_forward_output_over_its_input(shift):
    """The output may overlap the input: rows are then staged."""
    n = 100
    net, _, x, _ = _net(n, 7)
    buf = torch.zeros(12 * n + 8 * n, dtype=torch.float32, device="cuda")
    buf[shift:shift + 8 * n] = torch.from_numpy(x).cuda().ravel()
    ref = torch.empty((n, 12), dtype=torch.float32, device="cuda")
    net.forward(torch.from_numpy(x).cuda(), ref)
    for f in (net.forward, net.forward_noalloc):
        b = buf.clone()
        f(b[shift:shift + 8 * n].view(n, 8), b[:12 * n].view(n, 12))
        assert torch.equal(b[:12 * n].view(n, 12), ref)
    net.close()
