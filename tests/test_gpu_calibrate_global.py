"""Unfused global peak on both sides of two events per compute unit, where its
first stage stops asking for the next chunk ahead: a batch in one call equals
the same events in small calls."""
import numpy as np
import pytest

import dl0sim
import paper_1307_6489_amd as rta
from test_gpu_flagged_pixels import pulse_traces
from test_gpu_parity import say, to_dev, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_samp", [4, 8, 9, 25, 255])
def test_one_call_equals_small_calls(torch_dev, n_samp):
    import torch
    ct = dl0sim.CameraType("glob%d" % n_samp, 61, n_samp, 2, 16.0)
    rng = np.random.default_rng(n_samp)
    n = 2 * torch.cuda.get_device_properties(torch_dev).multi_processor_count + 60
    amps = np.where(rng.random((n, 61)) < 0.3, np.exp(rng.uniform(3.0, 9.0, (n, 61))), 0.0)
    tr = pulse_traces(ct, amps, s0=max(0, n_samp - 9))
    tr[..., :61] += rng.integers(0, 30, tr[..., :61].shape).astype(np.uint16)
    say("global peak: 61 x %d, %d events" % (n_samp, n))
    cam, d = rta.Camera.from_type(ct), to_dev(tr, torch_dev)
    whole = rta.calibrate(cam, d, extractor=rta.EXTRACT_GLOBAL_PEAK)
    for a in range(0, n, 100):
        part = rta.calibrate(cam, d[a:a + 100].contiguous(), extractor=rta.EXTRACT_GLOBAL_PEAK)
        for k, v in part.items():
            assert torch.equal(whole[k][a:a + 100], v), k
    assert whole["gain"].any() and len(torch.unique(whole["sstar"])) > (0 if n_samp == 4 else 1)
