"""Flagged pixels, islands and low-gain gathers of the fused kernel at the
edges of their per-wavefront rounds.

The fused kernel works on each wavefront's run of flagged pixels (D at or
above the boundary or picture threshold) 64 at a time, finds the islands of
images of at most 64 mask pixels by flood fill over slot masks, and gathers
the low-gain samples of a wavefront with few switched pixels instead of
streaming the gain again.  Every record is compared with the oracle.
"""
import numpy as np
import pytest

import dl0sim
import oracle
import paper_1307_6489_amd as rta
from test_gpu_parity import check_records, oracle_events, say, to_dev, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
PULSE = np.array([0.3, 1.0, 0.6, 0.2])
SCHEDULES = [(8, 4, 0, 8), (4, 8, 0, 8), (2, 4, 2, 16)]


def pulse_traces(ct, amps, s0=2):
    """uint16 [E][G][T][Npad]: the rounded pedestal plus a pulse of amps[e][i]
    high-gain ADC (1/16 of it in the low gain) in pixel i, four samples long."""
    E, N, G, T = len(amps), ct.n_pix, ct.n_gain, ct.n_samp
    tr = np.zeros((E, G, T, ct.n_pix_pad), np.uint16)
    for g in range(G):
        tr[:, g, :, :N] = np.rint(ct.ped[g]).astype(np.uint16)[None, None, :]
        a = np.asarray(amps, np.float64) / (1.0 if g == 0 else 16.0)
        at = np.minimum(s0 + (np.arange(N) % 3), T - 4)
        for k in range(4):
            add = np.rint(a * PULSE[k]).astype(np.int64)
            for e in range(E):
                v = tr[e, g, at + k, np.arange(N)].astype(np.int64) + add[e]
                tr[e, g, at + k, np.arange(N)] = np.minimum(v, 4095 if (G == 2 and g == 0) else 65535)
    return tr


def fused_against_oracle(ct, tr, dev, extractor=rta.EXTRACT_SLIDING, schedules=SCHEDULES):
    import torch
    E = len(tr)
    oc = oracle.Camera.from_type(ct, extractor=extractor)
    offs = np.arange(E, dtype=np.int64) * oc.event_elems
    pixes, masks, recs = oracle_events([oc], np.zeros(E, np.int64), tr.reshape(-1), offs)
    pipe = rta.Pipeline([rta.Camera.from_type(ct)], do_stereo=False, extractor=extractor)
    b = pipe.make_batch(to_dev(tr.reshape(-1), dev), torch.zeros(E, dtype=torch.int32, device=dev), to_dev(offs, dev))
    for sched in schedules:
        say("  schedule", sched)
        pipe.set_schedule(*sched)
        tel, _ = pipe.alloc_outputs(b, dev)
        tel.fill_(float("nan"))
        pipe.process(b, tel)
        check_records(rta.records(tel), recs, pixes, masks, lambda k: ct, "fused %s" % (sched,))
    assert pipe.status() == 0
    return pixes, masks, recs


@pytest.mark.parametrize("n_pix", [7, 64, 65, 1855, 2048])
def test_many_flagged_pixels(torch_dev, n_pix):
    """Boundary-level charge in up to every pixel (several rounds of 64 per
    wavefront) around a few picture pixels: masks from none to over 64."""
    ct = dl0sim.CameraType("flag%d" % n_pix, n_pix, 12, 1, 28.0)
    rng = np.random.default_rng(n_pix)
    amps = []
    for share in (0.02, 0.3, 0.7, 1.0):
        for n_pic in (0, 1, 4, 8, 30):
            a = np.where(rng.random(n_pix) < share, rng.uniform(42.0, 47.0, n_pix), 0.0)  # 9 to 10 p.e.: boundary only
            a[rng.permutation(n_pix)[:n_pic]] = rng.uniform(80.0, 900.0)
            amps.append(a)
    say("flagged pixels: %d px, %d events" % (n_pix, len(amps)))
    tr = pulse_traces(ct, amps)
    pixes, masks, recs = fused_against_oracle(ct, tr, torch_dev)
    n = [int(r["n_pix"]) for r in recs]
    if n_pix >= 1855:
        first = [int(((p["q"] >= 5.0)[:512]).sum()) for p in pixes]
        assert any(f > 128 and 0 < m <= 64 for f, m in zip(first, n))
        assert any(f > 128 and m > 64 for f, m in zip(first, n))


def test_islands_of_a_one_sided_neighbour_table(torch_dev):
    """Edges are taken from the row of the smaller pixel: with entries of the
    table removed at random, the fused and unfused island counts equal the
    connected components of those edges, in small and in large images."""
    import torch
    from scipy.sparse import coo_matrix
    from scipy.sparse.csgraph import connected_components
    ct = dl0sim.CameraType("onesided", 331, 12, 1, 28.0)
    rng = np.random.default_rng(3)
    nbr = ct.geom.nbr.copy()
    nbr[rng.random(nbr.shape) < 0.5] = -1
    cam = rta.Camera(ct.n_pix, ct.n_samp, 1, ct.geom.x, ct.geom.y, nbr, ct.ped, ct.adc_per_pe, ct.focal_m)
    amps = np.stack([np.where(rng.random(331) < share, 300.0, 0.0) for share in (0.05, 0.1, 0.15, 0.2, 0.3, 0.6, 0.9)])
    tr = pulse_traces(ct, amps)
    say("one-sided neighbour table: 331 px, %d events" % len(tr))
    out = rta.calibrate(cam, to_dev(tr, torch_dev))
    mask = rta.clean(cam, out["D"])
    unfused = rta.records(rta.hillas(cam, out["q"], out["t"], mask))
    pipe = rta.Pipeline([cam], do_stereo=False)
    E = len(tr)
    b = pipe.make_batch(to_dev(tr.reshape(-1), torch_dev), torch.zeros(E, dtype=torch.int32, device=torch_dev),
                        torch.arange(E, dtype=torch.int64, device=torch_dev) * cam.event_elems)
    tel, _ = pipe.alloc_outputs(b, torch_dev)
    pipe.process(b, tel)
    fused = rta.records(tel)
    m = mask.cpu().numpy().astype(bool)
    sizes = m.sum(1)
    assert sizes.min() <= 64 < sizes.max()
    for e in range(E):
        i, k = np.nonzero((nbr > np.arange(331)[:, None]) & m[e][:, None])
        j = nbr[i, k]
        ok = m[e][j]
        g = coo_matrix((np.ones(ok.sum()), (i[ok], j[ok])), shape=(331, 331))
        comp = connected_components(g, directed=False)[1]
        want = len(set(comp[m[e]].tolist()))
        assert int(fused["n_islands"][e]) == want == int(unfused["n_islands"][e])
        assert int(fused["n_pix"][e]) == sizes[e] == int(unfused["n_pix"][e])


@pytest.mark.parametrize("n_samp", [4, 25, 63, 64, 65, 128, 192, 193, 255])
def test_low_gain_pixels_per_wavefront(torch_dev, n_samp):
    """0 to 40 switched pixels in one wavefront's pixels (consecutive and one
    per lane), on both sides of the gather's limits of 4, 8 and 16."""
    ct = dl0sim.CameraType("low%d" % n_samp, 1855, n_samp, 2, 28.0)
    rng = np.random.default_rng(n_samp)
    amps = []
    for n in (0, 1, 2, 4, 5, 8, 9, 15, 16, 17, 40):
        for stride in (1, 8):
            a = np.zeros(1855)
            at = (7 + stride * np.arange(n)) if stride == 1 else 512 + stride * np.arange(n)
            a[at] = rng.uniform(3.8e3, 6.0e4, n)
            a[1854] = 5000.0 if n % 2 else 0.0
            amps.append(a)
    say("low-gain pixels: 1855 x %d, %d events" % (n_samp, len(amps)))
    tr = pulse_traces(ct, amps, s0=max(0, n_samp - 9))
    # a late, lower maximum and noise in the low gain, so that its windows differ from the high gain's
    tr[:, 1, : n_samp // 2, :1855] += rng.integers(0, 40, (len(tr), n_samp // 2, 1855)).astype(np.uint16)
    _, _, recs = fused_against_oracle(ct, tr, torch_dev)
    assert max(int(r["n_lowgain"]) for r in recs) >= 40
