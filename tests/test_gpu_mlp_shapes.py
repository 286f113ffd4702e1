"""Training passes at the shapes where their kernels change: every width (64 .. 512),
one hidden layer (no hidden map) and several, batches up to and past the line between
workgroups of 32 and 64 rows (64 rows a compute unit), forward passes that end inside a
workgroup.  The gradient and
the forward pass of a batch must equal, to rounding, those of the
FP64 reference with the device's BF16 weights; the bound, on each map's 2-norm, is that
of the BF16 rounding of the stored activations and gradients: 2^-8 a stored value, at
most 2 (L + 1) of them in a chain."""
import numpy as np
import pytest

from oracle import mlp as ref

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,hidden,batch", [(64, 1, 64), (64, 2, 128), (128, 3, 192), (192, 2, 64), (256, 4, 1984),
                                                (320, 2, 192), (384, 3, 128), (448, 2, 192), (512, 3, 64),
                                                (64, 3, 16320), (64, 3, 16384), (128, 2, 16448)])
def test_gradient_shapes(width, hidden, batch):
    import torch
    from paper_1908_05662_amd.api import Convolver, Mlp

    say(f"case: training pass {width} x {hidden}, {batch} rows")
    rng = np.random.default_rng(width + hidden + batch)
    v = rng.normal(size=(batch, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    psi = rng.uniform(0, 2 * np.pi, batch)
    x = np.concatenate([v, np.sin(psi)[:, None], np.cos(psi)[:, None]], 1).astype(np.float32)
    t = rng.normal(size=(batch, 3)).astype(np.float32)
    conv = Convolver(0)
    m = Mlp(conv, width, hidden, max_batch=batch, seed=7)
    p = m.get_params().numpy().astype(np.float64)
    x64, t64 = x.astype(np.float64), t.astype(np.float64)
    tol = 2 * (hidden + 1) * 2.0**-8
    xt, tt = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y, _ = ref.forward(p, x64, width, hidden)
    for n in (batch, batch - 7, 1):
        got = m.forward(xt[:n]).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - y[:n]) <= tol * np.linalg.norm(y[:n]), n
    loss, g = m.gradient(xt, tt)
    loss2, g2 = m.gradient(xt, tt)
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
    want_loss, want = ref.loss_and_grad(p, x64, t64, width, hidden)
    assert abs(loss.item() - want_loss) <= tol * want_loss
    g = g.cpu().numpy().astype(np.float64)
    lay, _ = ref.layout(width, hidden)
    for l, (wo, r, c, bo) in enumerate(lay):
        for name, o, k in (("weights", wo, r * c), ("biases", bo, r)):
            e = np.linalg.norm(g[o:o + k] - want[o:o + k]) / np.linalg.norm(want[o:o + k])
            assert e <= tol, (l, name, e)
    m.close()
    conv.close()
