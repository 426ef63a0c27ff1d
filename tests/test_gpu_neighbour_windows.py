"""The fused neighbour peak's windows, formed only for the pixels that can
enter the image, against the full scan of the unfused calibration and the
oracle.

The fused kernel bounds every pixel's window sum by its own sliding maximum,
asks for the neighbour windows of the pixels that the bounds' mask holds, and
stages their traces as many slices at once as fit; with more than 512 pixels
asked or 600 traces needed it scans every pixel.  The full scan forms sums in
saturating 16-bit halves and repeats an event in 32 bits when one may not
have fitted; high pedestals go to 32 bits at once.
"""
import numpy as np
import pytest

import dl0sim
import paper_1307_6489_amd as rta
from test_gpu_flagged_pixels import fused_against_oracle, pulse_traces
from test_gpu_parity import say, to_dev, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
NBR = rta.EXTRACT_NEIGHBOUR_PEAK
SCHEDULES = [(8, 4, 0, 8), (4, 8, 0, 16), (2, 4, 0, 8)]


def noisy(ct, tr, seed, sigma=6):
    rng = np.random.default_rng(seed)
    v = tr[:, :, :, :ct.n_pix].astype(np.int64) + rng.integers(-sigma, sigma + 1, tr[:, :, :, :ct.n_pix].shape)
    tr[:, :, :, :ct.n_pix] = np.clip(v, 0, 65535)
    if ct.n_gain == 2:
        tr[:, 0] = np.minimum(tr[:, 0], 4095)
    tr[:, :, :, ct.n_pix:] = 65535  # padding pixels are ignored
    return tr


def against_full_scan(ct, tr, dev, cam=None):
    """Fused records against calibrate (every pixel scanned) -> clean -> hillas."""
    import torch
    cam = cam or rta.Camera.from_type(ct)
    E = len(tr)
    out = rta.calibrate(cam, to_dev(tr, dev), extractor=NBR)
    mask = rta.clean(cam, out["D"], out["gain"])
    want = rta.hillas(cam, out["q"], out["t"], mask, out["gain"]).cpu()
    pipe = rta.Pipeline([cam], do_stereo=False, extractor=NBR)
    b = pipe.make_batch(to_dev(tr.reshape(-1), dev), torch.zeros(E, dtype=torch.int32, device=dev),
                        torch.arange(E, dtype=torch.int64, device=dev) * cam.event_elems)
    tel, _ = pipe.alloc_outputs(b, dev)
    tel.fill_(float("nan"))
    pipe.process(b, tel)
    same = [k for k in range(16) if k not in (8, 9)]
    assert torch.equal(tel.cpu().view(torch.int32)[:, same], want.view(torch.int32)[:, same])
    return rta.records(tel)


@pytest.mark.parametrize("n_pix", [1, 7, 61, 1764, 2048])
def test_asked_pixels(torch_dev, n_pix):
    """No pixel to every pixel asked, on both sides of the 512 and 600 limits."""
    ct = dl0sim.CameraType("ask%d" % n_pix, n_pix, 20, 1, 28.0)
    rng = np.random.default_rng(n_pix)
    near = np.argsort(ct.geom.x.astype(np.float64) ** 2 + ct.geom.y.astype(np.float64) ** 2 * 1.7)
    amps = []
    for n in (0, 1, 2, 5, 40, 64, 65, 130, 400, 500, 512, 530, 600, 2048):
        a = np.zeros(n_pix)
        a[near[:n]] = rng.uniform(60.0, 900.0, min(n, n_pix))
        amps.append(a)
    amps.append(np.where(rng.random(n_pix) < 0.2, rng.uniform(60.0, 200.0, n_pix), 0.0))
    say("neighbour windows: %d px, %d events" % (n_pix, len(amps)))
    tr = noisy(ct, pulse_traces(ct, amps, s0=6), n_pix)
    _, _, recs = fused_against_oracle(ct, tr, torch_dev, NBR, SCHEDULES)
    got = against_full_scan(ct, tr, torch_dev)
    if n_pix >= 1764:
        n = np.array([int(r["n_pix"]) for r in recs])
        assert (n == 0).any() and ((n > 0) & (n <= 64)).any() and ((n > 64) & (n <= 512)).any() and (n > 600).any()
    assert [int(v) for v in got["n_pix"]] == [int(r["n_pix"]) for r in recs]


@pytest.mark.parametrize("n_samp", [4, 5, 7, 8, 25, 40, 65, 128, 255])
def test_trace_lengths(torch_dev, n_samp):
    """One to many stages of slices, dual gain with switched pixels."""
    ct = dl0sim.CameraType("len%d" % n_samp, 1855, n_samp, 2, 28.0)
    rng = np.random.default_rng(n_samp)
    x, y = ct.geom.x.astype(np.float64), ct.geom.y.astype(np.float64)
    amps = []
    for n in (3, 20, 50, 90, 200, 450):
        d = np.hypot(x - rng.uniform(-0.5, 0.5), (y - rng.uniform(-0.5, 0.5)) * 2.0)
        a = np.zeros(1855)
        a[np.argsort(d)[:n]] = np.exp(rng.uniform(np.log(60.0), np.log(3.0e4), n))
        amps.append(a)
    say("neighbour windows: 1855 x %d, %d events" % (n_samp, len(amps)))
    tr = noisy(ct, pulse_traces(ct, amps, s0=max(0, n_samp // 2 - 4)), n_samp)
    _, _, recs = fused_against_oracle(ct, tr, torch_dev, NBR, SCHEDULES)
    against_full_scan(ct, tr, torch_dev)
    assert max(int(r["n_lowgain"]) for r in recs) > 20


@pytest.mark.parametrize("ped", [300.0, 2000.0, 2040.0, 2060.0, 9000.0])
def test_sums_around_sixteen_bits(torch_dev, ped):
    """Neighbour sums of up to 24 samples on both sides of 65535, from the
    signal and from the pedestal alone (49152 / 24 = 2048 ADC)."""
    ct = dl0sim.CameraType("sat", 331, 30, 1, 28.0, base_pedestal=ped)
    amps = np.zeros((8, 331))
    for k, v in enumerate((500.0, 2.0e3, 3.0e3, 4.0e3, 8.0e3, 2.0e4, 4.0e4, 5.5e4)):
        amps[k, :60] = v
    tr = noisy(ct, pulse_traces(ct, amps, s0=9), int(ped))
    say("16-bit neighbour sums: pedestal %g" % ped)
    fused_against_oracle(ct, tr, torch_dev, NBR, SCHEDULES)
    against_full_scan(ct, tr, torch_dev)


@pytest.mark.parametrize("levels", [(10.0, 5.0), (3.0, 1.0), (1.0, 0.0), (0.0, -5.0)])
def test_levels_and_one_sided_neighbours(torch_dev, levels):
    """Cleaning levels down to below zero (every pixel needed), and neighbour
    tables with entries removed at random."""
    ct = dl0sim.CameraType("lev", 397, 24, 2, 28.0)
    rng = np.random.default_rng(8)
    amps = np.where(rng.random((10, 397)) < 0.15, rng.uniform(40.0, 400.0, (10, 397)), 0.0)
    amps[0] = 0.0
    tr = noisy(ct, pulse_traces(ct, amps, s0=8), 5)
    for cut in (0.0, 0.5):
        nbr = ct.geom.nbr.copy()
        nbr[rng.random(nbr.shape) < cut] = -1
        cam = rta.Camera(ct.n_pix, ct.n_samp, 2, ct.geom.x, ct.geom.y, nbr, ct.ped, ct.adc_per_pe, ct.focal_m,
                         t_pic=levels[0], t_bnd=levels[1])
        say("neighbour windows: levels %s, %d%% of neighbours removed" % (levels, 100 * cut))
        against_full_scan(ct, tr, torch_dev, cam)
