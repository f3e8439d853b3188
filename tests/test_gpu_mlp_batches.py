"""The network's gradient at the edges of its chunks (128 samples) and sample
tiles (16), against the fp64 oracle.

Bar, per entry: a gradient entry is a sum over the batch of products of
rounded factors.  With u = 2^-24, every factor carries at most the rounding of
the sums before it (16 + 64 + 64 + 64 + 3 terms, the tanh and elementwise
steps: under 300 u of the sums of absolute values), and the sum over the batch
adds batch u: |error| <= (batch + 300) u G, G the same gradient with every
sum replaced by the sum of absolute values."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mlp as OM
from paper_2109_01232_amd import binding as B

from gpu_common import dev_tensor, say

pytestmark = pytest.mark.gpu


def absolute_gradient(p, X, T, shift, scale):
    """Sums of absolute values along the gradient's own path (tanh' <= 1)."""
    (W1, b1), (W2, b2), (W3, b3) = OM.unpack(p)
    X = np.abs((X - shift) * scale)
    h1 = np.minimum(1.0, X @ np.abs(W1) + np.abs(b1))
    h2 = np.minimum(1.0, h1 @ np.abs(W2) + np.abs(b2))
    dy = 2.0 * (h2 @ np.abs(W3) + np.abs(b3) + np.abs(T)) / T.size
    d2 = dy @ np.abs(W3).T
    d1 = d2 @ np.abs(W2).T
    return OM.pack([(X.T @ d1, d1.sum(0)), (h1.T @ d2, d2.sum(0)), (h2.T @ dy, dy.sum(0))])


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 127, 128, 129, 256, 1000])
def test_gradient_at_chunk_edges(batch):
    rng = np.random.default_rng(batch)
    c = lambda a: np.asarray(a, dtype=np.float32)
    p = c(OM.init_params(batch) + rng.normal(0, 0.05, OM.NPARAM))
    X, T = c(rng.standard_normal((batch, 16)) * 2 + 1), c(rng.standard_normal((batch, 3)))
    shift, scale = c(rng.standard_normal(16)), c(rng.uniform(0.2, 1.0, 16))
    g = torch.full((OM.NPARAM,), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    say("mlp gradient, batch", batch)
    B.gmresir_mlp_loss_grad(*(dev_tensor(a) for a in (p, shift, scale, X, T)), g, loss)
    d = [a.astype(np.float64) for a in (p, X, T, shift, scale)]
    lref, gref = OM.loss_and_grad(*d)
    u = 2.0 ** -24
    G = absolute_gradient(*d)
    assert np.all(np.abs(g.cpu().numpy() - gref) <= (batch + 300) * u * G)
    assert abs(loss.item() - lref) <= 1e-5 * lref
    # one Adam step on the same batch takes this gradient: first moments 0.1 g
    P_, m, v = dev_tensor(p), torch.zeros_like(g), torch.zeros_like(g)
    B.gmresir_mlp_train_step(P_, m, v, *(dev_tensor(a) for a in (shift, scale, X, T)), 1e-3, 1, loss)
    assert torch.equal(m, (1.0 - torch.tensor(0.9)).cuda() * g)
