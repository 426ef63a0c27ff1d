"""Every way through the fused neighbour peak gives the full scan's bits: small
cameras scanned, bounds given up after one chunk under a noisy start of the
trace, windows up to the limit of traces and the scan past it."""
import numpy as np
import pytest

import dl0sim
import paper_1307_6489_amd as rta
from test_gpu_flagged_pixels import fused_against_oracle, pulse_traces
from test_gpu_neighbour_windows import against_full_scan, noisy
from test_gpu_parity import say, to_dev, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
NBR = rta.EXTRACT_NEIGHBOUR_PEAK
SCHEDULES = [(8, 4, 0, 8), (8, 8, 0, 16), (4, 8, 0, 16), (2, 4, 0, 8)]


@pytest.mark.parametrize("n_pix,n_samp", [(959, 20), (960, 20), (1764, 15), (1764, 16), (1855, 40), (2048, 64), (2048, 70)])
def test_share_of_pixels_at_the_boundary(torch_dev, n_pix, n_samp):
    """0 to 60 % of the pixels at the boundary level in the first chunk (a few
    of them at the picture level), then an image; and images of 20 to 600 traces."""
    ct = dl0sim.CameraType("rule%d_%d" % (n_pix, n_samp), n_pix, n_samp, 2, 28.0)
    rng = np.random.default_rng(n_pix + n_samp)
    near = np.argsort(np.hypot(ct.geom.x.astype(np.float64), ct.geom.y.astype(np.float64) * 1.5))
    parts = []
    for share in (0.0, 0.03, 0.08, 0.12, 0.18, 0.3, 0.6):
        a = np.where(rng.random(n_pix) < share, rng.uniform(32.0, 47.0, n_pix), 0.0)
        a[rng.random(n_pix) < 0.02 * share] = 120.0
        b = np.zeros(n_pix)
        b[near[:40]] = np.exp(rng.uniform(np.log(60.0), np.log(2.0e4), 40))
        early = pulse_traces(ct, [a], s0=0).astype(np.int64)
        late = pulse_traces(ct, [b], s0=n_samp - 7).astype(np.int64) - pulse_traces(ct, [np.zeros(n_pix)])
        parts.append(np.minimum(early + late, 65535).astype(np.uint16))
    for n in (3, 60, 150, 200, 230, 260, 300, 330, 500):
        b = np.zeros(n_pix)
        b[near[:n]] = rng.uniform(60.0, 900.0, n)
        parts.append(pulse_traces(ct, [b], s0=n_samp - 7))
    tr = noisy(ct, np.concatenate(parts), n_pix)
    say("neighbour rule: %d x %d, %d events" % (n_pix, n_samp, len(tr)))
    _, _, recs = fused_against_oracle(ct, tr, torch_dev, NBR, SCHEDULES)
    got = against_full_scan(ct, tr, torch_dev)
    assert [int(v) for v in got["n_pix"]] == [int(r["n_pix"]) for r in recs]
    n = [int(r["n_pix"]) for r in recs]
    assert min(n) < 10 and max(n) > 300
    # more than two telescopes per compute unit: the share is looked at
    import torch
    E, d = len(tr), to_dev(tr.reshape(-1), torch_dev)
    n_tel = 2 * torch.cuda.get_device_properties(torch_dev).multi_processor_count + E
    at = torch.arange(n_tel, device=torch_dev) % E
    pipe = rta.Pipeline([rta.Camera.from_type(ct)], do_stereo=False, extractor=NBR)
    few = pipe.make_batch(d, torch.zeros(E, dtype=torch.int32, device=torch_dev), at[:E] * (d.numel() // E))
    many = pipe.make_batch(d, torch.zeros(n_tel, dtype=torch.int32, device=torch_dev), at * (d.numel() // E))
    for sched in SCHEDULES:
        say("  schedule", sched)
        pipe.set_schedule(*sched)
        a, b = pipe.alloc_outputs(few, torch_dev)[0], pipe.alloc_outputs(many, torch_dev)[0]
        pipe.process(few, a)
        pipe.process(many, b)
        same = [k for k in range(16) if k not in (8, 9)]
        assert torch.equal(a[at][:, same].view(torch.int32), b[:, same].view(torch.int32))
