"""Neighbour sums that leave 16 bits anywhere in a trace: the scan goes on in 32
bits from there, for the wavefront alone, in the unfused calibration and in the
fused kernel (which scans every pixel at low picture levels), against the
oracle.  With a pedestal of 300 a window of 24 samples reaches 65535 at pulses of
about 4630 ADC."""
import numpy as np
import pytest

import dl0sim
import oracle
import paper_1307_6489_amd as rta
from test_gpu_extractors import calib_parity
from test_gpu_flagged_pixels import pulse_traces
from test_gpu_parity import check_records, oracle_events, say, to_dev, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
NBR = rta.EXTRACT_NEIGHBOUR_PEAK


def bright(n_pix, n_samp, ped, seed):
    """Pulses around the limit at every phase of the four staged slices, in few
    pixels and in all, then an earlier or later brighter one in some events."""
    ct = dl0sim.CameraType("sum%d_%d" % (n_pix, n_samp), n_pix, n_samp, 1, 28.0, base_pedestal=ped)
    rng = np.random.default_rng(seed)
    r = np.hypot(ct.geom.x.astype(np.float64) - 0.2, ct.geom.y.astype(np.float64))
    near = np.argsort(r)
    out = []
    for k, (amp, n) in enumerate(((3000.0, 40), (4500.0, 60), (4620.0, 60), (4640.0, 60), (4700.0, n_pix), (9.0e3, 12),
                                  (3.0e4, 30), (6.0e4, n_pix), (2.0e4, 1))):
        a = np.zeros(n_pix)
        a[near[:n]] = amp * rng.uniform(0.98, 1.02, min(n, n_pix))
        tr = pulse_traces(ct, [a], s0=int(rng.integers(0, max(1, n_samp - 6))))
        if k % 2:
            b = np.zeros(n_pix)
            b[near[n_pix // 2:n_pix // 2 + 30]] = rng.uniform(2.0e3, 5.0e4)
            second = pulse_traces(ct, [b], s0=int(rng.integers(0, max(1, n_samp - 6)))).astype(np.int64)
            tr = np.minimum(tr + second - pulse_traces(ct, [np.zeros(n_pix)]), 65535).astype(np.uint16)
        out.append(tr)
    tr = np.concatenate(out)
    v = tr[..., :n_pix].astype(np.int64) + rng.integers(-6, 7, tr[..., :n_pix].shape)
    tr[..., :n_pix] = np.clip(v, 0, 65535)
    tr[..., n_pix:] = 65535  # padding pixels are ignored
    return ct, tr


@pytest.mark.parametrize("ped", [300.0, 2725.0, 2731.0, 20000.0])
@pytest.mark.parametrize("n_pix,n_samp", [(331, 4), (331, 7), (1855, 25), (2048, 64)])
def test_sums_past_sixteen_bits(torch_dev, n_pix, n_samp, ped):
    import torch
    ct, tr = bright(n_pix, n_samp, ped, n_samp + int(ped))
    say("neighbour sums: %d x %d, pedestal %g" % (n_pix, n_samp, ped))
    calib_parity(ct, tr, torch_dev, NBR)
    # picture level below 5 p.e.: every pixel is scanned
    E, levels = len(tr), dict(t_pic=4.0, t_bnd=2.0)
    oc = oracle.Camera.from_type(ct, extractor=NBR, **levels)
    offs = np.arange(E, dtype=np.int64) * oc.event_elems
    pixes, masks, recs = oracle_events([oc], np.zeros(E, np.int64), tr.reshape(-1), offs)
    cam = rta.Camera(ct.n_pix, ct.n_samp, 1, ct.geom.x, ct.geom.y, ct.geom.nbr, ct.ped, ct.adc_per_pe, ct.focal_m, **levels)
    pipe = rta.Pipeline([cam], do_stereo=False, extractor=NBR)
    b = pipe.make_batch(to_dev(tr.reshape(-1), torch_dev), torch.zeros(E, dtype=torch.int32, device=torch_dev), to_dev(offs, torch_dev))
    for sched in ((8, 4, 0, 8), (4, 8, 0, 16)):
        pipe.set_schedule(*sched)
        tel, _ = pipe.alloc_outputs(b, torch_dev)
        tel.fill_(float("nan"))
        pipe.process(b, tel)
        check_records(rta.records(tel), recs, pixes, masks, lambda k: ct, "fused %s" % (sched,))
