"""The network's row tiles and batch slices at their edges: wavefronts that
take several tiles in turn, partial tiles and slices of the weight-gradient
contraction, the loss sum's rounds of 2048 rows."""
import numpy as np
import pytest

import paper_1307_6489_amd as rta
from test_gpu_event_pass import network
from test_gpu_parity import say, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
LAYERS = ((10, 64), (64, 64), (64, 64), (64, 2))


def batch(B, dev):
    import torch
    g = torch.Generator().manual_seed(B)
    x = torch.randn((B, 10), generator=g) + 0.1
    return x.to(dev), (torch.rand(B, generator=g) > 0.4).float().to(dev), torch.randn(B, generator=g).to(dev)


@pytest.mark.parametrize("B", [49151, 49152, 49153, 70001])
def test_forward_tiles_in_turn(torch_dev, B):
    import torch
    m, _ = network()
    x, _, _ = batch(B, torch_dev)
    say("forward: %d rows" % B)
    whole = m.forward(x)
    parts = torch.cat([m.forward(x[a:a + 1009].contiguous()) for a in range(0, B, 1009)])
    assert torch.equal(whole.view(torch.int32), parts.view(torch.int32))


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 65, 255, 256, 257, 1040, 2047, 2048, 2049, 4096, 4097, 4400])
def test_gradient_slices(torch_dev, B):
    """Gradients from the stored bfloat16 activations and signals: each is a
    float32 sum of B exact products, within (B + 16) 2^-23 sum |terms| of the
    exact value for any order of the additions."""
    base, _ = network()
    m = rta.Mlp(max_batch=4400)
    m.set_params(base.get_params(), np.zeros(10, np.float32) + 0.1, np.ones(10, np.float32))
    x, label, log10e = batch(B, torch_dev)
    say("gradient: %d rows" % B)
    loss, grad = m.loss_grad(x, label, log10e)
    grad = grad.cpu().numpy().astype(np.float64)
    H = [m.stored(k, B).astype(np.float64) for k in range(4)]
    G = [m.stored(k, B).astype(np.float64) for k in (4, 5, 6, 7)]
    at = 0
    for (n_in, n_out), h, g in zip(LAYERS, H, G):
        for want, bound in ((h[:n_in] @ g[:n_out].T, np.abs(h[:n_in]) @ np.abs(g[:n_out]).T),
                            (g[:n_out].sum(1), np.abs(g[:n_out]).sum(1))):
            got = grad[at:at + want.size].reshape(want.shape)
            assert np.all(np.abs(got - want) <= (B + 16) * 2.0 ** -23 * bound + 1e-30)
            at += want.size
    o = m.forward(x).cpu().numpy().astype(np.float64)
    lab, y = label.cpu().numpy().astype(np.float64), log10e.cpu().numpy().astype(np.float64)
    rows = np.maximum(o[:, 0], 0) - o[:, 0] * lab + np.log1p(np.exp(-np.abs(o[:, 0]))) + lab * (o[:, 1] - y) ** 2
    terms = np.abs(o[:, 0]) * (1 + lab) + 1 + lab * (np.abs(o[:, 1]) + np.abs(y)) ** 2  # a row's own roundings
    assert abs(float(loss) - rows.mean()) <= 2.0 ** -23 * ((B / 64 + 12) * rows.sum() + 16 * terms.sum()) / B
