"""Calls that read their results back, on a stream given by the caller that is
still busy: they wait for that stream, not for the current one."""
import numpy as np
import pytest

import dl0sim
import paper_1307_6489_amd as rta
from test_gpu_parity import say, to_dev, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def busy(stream, dev):
    """Some ten milliseconds of work ahead of what follows on the stream."""
    import torch
    with torch.cuda.stream(stream):
        x = torch.ones((4096, 4096), device=dev)
        for _ in range(20):
            x = x @ x * 1e-4
    return x


def test_alert_search(torch_dev):
    import torch
    rng = np.random.default_rng(1)
    n = 20000
    e = np.zeros(n, rta.EVENT_DTYPE)
    e["dir_x"], e["dir_y"] = rng.uniform(-0.04, 0.04, n), rng.uniform(-0.04, 0.04, n)
    e["dir_x"][:300], e["dir_y"][:300] = 0.01, 0.004
    e["gammaness"] = 0.9
    evt, t = to_dev(e.view(np.float32).reshape(n, -1), torch_dev), to_dev(rng.uniform(0.0, 100.0, n), torch_dev)
    sam = rta.Sam(48, 100, 0.0, 1.0, 0.002, 1.5, 3.5, 7.0, 0.7, 5.0, [1, 10, 100])
    sam.fill(evt, t)
    want = sam.search(99)
    torch.cuda.synchronize()
    assert want[4] > 0
    side = torch.cuda.Stream()
    for _ in range(3):
        keep = busy(side, torch_dev)
        say("alert search behind a busy stream")
        got = sam.search(99, stream=side)
        assert got[4] == want[4] and np.array_equal(got[3], want[3])
        for a, b in zip(got[:3], want[:3]):
            assert torch.equal(a, b)
        del keep


class Pointer:
    """A stream known by its pointer alone."""

    def __init__(self, stream):
        self.cuda_stream = stream.cuda_stream


@pytest.mark.parametrize("wrap", [lambda s: s, Pointer])
def test_health_on_the_default_stream_from_another(torch_dev, wrap):
    import torch
    ct = dl0sim.CameraType("default", 61, 16, 1, 28.0)
    tr = np.random.default_rng(4).integers(280, 330, (40, 1, 16, ct.n_pix_pad)).astype(np.uint16)
    cam, d = rta.Camera.from_type(ct), to_dev(tr, torch_dev)
    pix, out = rta.health(cam, d)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for given in (torch.cuda.default_stream(), torch.cuda.Stream()):
            keep = busy(given, torch_dev)
            say("health on a busy stream, from another")
            p2, o2 = rta.health(cam, d, stream=wrap(given))
            assert np.array_equal(p2, pix) and np.array_equal(o2, out)
            del keep


def test_health(torch_dev):
    import torch
    ct = dl0sim.CameraType("stream", 331, 16, 1, 28.0)
    rng = np.random.default_rng(2)
    tr = rng.integers(280, 330, (40, 1, 16, ct.n_pix_pad)).astype(np.uint16)
    cam, d = rta.Camera.from_type(ct), to_dev(tr, torch_dev)
    pix, out = rta.health(cam, d)
    side = torch.cuda.Stream()
    for _ in range(3):
        keep = busy(side, torch_dev)
        say("health behind a busy stream")
        p2, o2 = rta.health(cam, d, stream=side)
        assert np.array_equal(p2, pix) and np.array_equal(o2, out)
        del keep


def test_stored_activations(torch_dev):
    import torch
    rng = np.random.default_rng(3)
    net = rta.Mlp(256)
    net.set_params((0.1 * rng.standard_normal(rta.MLP_N_PARAMS)).astype(np.float32), np.zeros(10, np.float32),
                   np.ones(10, np.float32))
    x = to_dev(rng.standard_normal((256, 10)).astype(np.float32), torch_dev)
    y, e = to_dev((rng.random(256) < 0.5).astype(np.float32), torch_dev), to_dev(rng.random(256).astype(np.float32), torch_dev)
    net.loss_grad(x, y, e)
    want = net.stored(1, 256)
    side = torch.cuda.Stream()
    for _ in range(3):
        keep = busy(side, torch_dev)
        say("stored activations behind a busy stream")
        assert np.array_equal(net.stored(1, 256, stream=side), want)
        del keep
