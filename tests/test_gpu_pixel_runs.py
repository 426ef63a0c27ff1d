"""Runs of flagged pixels longer than 256 in the schedules with 8 pixels per
lane and 8 wavefronts, whose first four wavefronts extract 512 pixels each:
no flagged pixel is lost, with every extractor, against the oracle."""
import numpy as np
import pytest

import dl0sim
import paper_1307_6489_amd as rta
from test_gpu_flagged_pixels import fused_against_oracle, pulse_traces
from test_gpu_parity import say, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extractor", [rta.EXTRACT_SLIDING, rta.EXTRACT_FIXED, rta.EXTRACT_GLOBAL_PEAK,
                                       rta.EXTRACT_NEIGHBOUR_PEAK])
@pytest.mark.parametrize("n_pix", [600, 1855, 2048])
def test_long_runs(torch_dev, n_pix, extractor):
    ct = dl0sim.CameraType("run%d" % n_pix, n_pix, 12, 1, 28.0)
    rng = np.random.default_rng(n_pix)
    amps = []
    for lo, hi, share in ((0, 512, 0.6), (0, 600, 1.0), (256, 1100, 0.7), (512, 1536, 0.9), (0, 2048, 0.8), (0, 2048, 1.0)):
        for n_pic in (3, 40):
            a = np.where(rng.random(n_pix) < share, rng.uniform(42.0, 47.0, n_pix), 0.0)  # 9 to 10 p.e.: boundary only
            a[:lo] = a[hi:] = 0.0
            a[np.flatnonzero(a)[rng.permutation((a > 0).sum())[:n_pic]] if a.any() else []] = rng.uniform(80.0, 900.0)
            amps.append(a)
    say("long runs: %d px, extractor %d, %d events" % (n_pix, extractor, len(amps)))
    tr = pulse_traces(ct, amps)
    schedules = [(8, 8, 0, 8), (8, 8, 0, 16)]
    if extractor == rta.EXTRACT_SLIDING:
        schedules += [(8, 8, 1, 8), (8, 8, 2, 16)]
    pixes, _, recs = fused_against_oracle(ct, tr, torch_dev, extractor, schedules)
    if extractor == rta.EXTRACT_SLIDING:
        flagged = np.array([[int((p["q"][b:b + 512] >= 5.0).sum()) for b in range(0, n_pix, 512)] for p in pixes])
        assert (flagged[:, :-1] > 256).any() and (flagged[:, :-1] > 500).any()
    assert any(int(r["n_pix"]) > 0 for r in recs)
