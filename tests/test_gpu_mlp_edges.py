"""Training step of the rank network at odd batches (two samples per forward
block, a quarter of the batch per gradient wave) and with inputs that are
only float-aligned, against torch autograd in float64."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import get_rcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return get_rcs()


@pytest.mark.parametrize("batch", [1, 2, 3, 5, 31, 257])
@pytest.mark.parametrize("shift", [0, 1])
def test_backward_edges(env, batch, shift):
    rcs, torch = env
    g = inputs.rng(batch)
    wh = inputs.mlp_init(4).astype(np.float32)
    xh = g.random((batch, 66)).astype(np.float32)
    yh = g.standard_normal((batch, 32)).astype(np.float32)

    def place(a):      # `shift` floats past an aligned address
        buf = torch.zeros(a.size + shift, dtype=torch.float32, device="cuda")
        buf[shift:] = torch.from_numpy(a.reshape(-1)).cuda()
        return buf[shift:].reshape(a.shape)
    w, x, y = place(wh), place(xh), place(yh)
    grad, loss = place(np.zeros_like(wh)), place(np.zeros(1, np.float32))
    out = place(np.zeros((batch, 32), np.float32))
    rcs.mlp_backward(w, x, y, grad, loss)
    rcs.mlp_forward(w, x, out)
    W = torch.from_numpy(wh).double().requires_grad_(True)
    h, o = torch.from_numpy(xh).double(), 0
    for i, (fo, fi) in enumerate([(128, 66), (128, 128), (32, 128)]):
        h = h @ W[o:o + fo * fi].reshape(fo, fi).T + W[o + fo * fi:o + fo * fi + fo]
        o += fo * fi + fo
        h = torch.relu(h) if i < 2 else h
    L = ((h - torch.from_numpy(yh).double()) ** 2).mean()
    G, = torch.autograd.grad(L, W)
    # fp32 inner products of at most 128 (forward, deltas) and batch terms,
    # each a few units of 2^-24 sqrt(terms) of the row's norm
    assert np.allclose(out.cpu().numpy(), h.detach().numpy(), rtol=0, atol=2e-5)
    assert abs(loss.item() - L.item()) <= 2e-5 * L.item()
    assert np.linalg.norm(grad.cpu().numpy() - G.numpy()) <= 2e-5 * np.linalg.norm(G.numpy())
