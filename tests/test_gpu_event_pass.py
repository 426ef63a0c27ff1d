"""The per-event pass with the network, few and many array events.

Up to two events per compute unit take a workgroup each, its wavefronts on
the event's 16-telescope tiles; more events go to persistent wavefronts.
Both forms give the same bits, and the size-weighted means equal those of
rta_classify's rows up to float32 summation."""
import numpy as np
import pytest

import paper_1307_6489_amd as rta
from test_gpu_parity import say, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
MULT = [0, 1, 2, 15, 16, 17, 32, 33, 48, 63, 64, 65, 80, 130]


def make(dev, n_evt):
    import torch
    rng = np.random.default_rng(5)
    mult = np.array([MULT[k % len(MULT)] for k in range(n_evt)])
    off = np.zeros(n_evt + 1, np.int64)
    off[1:] = np.cumsum(mult)
    n = int(off[-1])
    rec = np.zeros(n, rta.HILLAS_DTYPE)
    rec["size"] = 10.0 ** rng.uniform(1.0, 5.0, n)     # some outside the trained range: box cuts
    rec["length"], rec["width"] = rng.uniform(0.02, 0.3, n), rng.uniform(0.01, 0.1, n)
    rec["cog_x"], rec["cog_y"] = rng.uniform(-0.8, 0.8, n), rng.uniform(-0.8, 0.8, n)
    rec["cog_dist"] = np.hypot(rec["cog_x"], rec["cog_y"])
    rec["psi"], rec["skewness"], rec["kurtosis"] = rng.uniform(-1.5, 1.5, n), rng.normal(0, 0.4, n), rng.normal(2.4, 0.4, n)
    rec["time_gradient"], rec["leakage"] = rng.normal(0, 3, n), rng.uniform(0, 0.5, n)
    rec["n_pix"], rec["n_islands"] = 20, rng.integers(1, 4, n)
    bad = rng.random(n) < 0.1
    rec["flags"][bad] = rta.FLAG_HILLAS_INVALID | rta.FLAG_TIME_INVALID
    ty = rng.integers(0, 2, n).astype(np.int32)
    ty[rng.random(n) < 0.02] = -1
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    return rec, ty, off, t(rec.view(np.float32).reshape(-1, 16)), t(ty), t(off)


def network():
    rng = np.random.default_rng(2)
    p = np.concatenate([v.ravel() for n_in, n_out in ((10, 64), (64, 64), (64, 64), (64, 2))
                        for v in (rng.normal(0, np.sqrt(2.0 / n_in), (n_in, n_out)), rng.normal(0, 0.1, n_out))])
    m = rta.Mlp(64)
    m.set_params(p.astype(np.float32), np.array([3, .1, .05, .5, 0, 0, 2.4, 0, .1, 1], np.float32),
                 np.array([1, .06, .03, .3, .9, .4, .5, 3, .2, 1], np.float32))
    bc = rta.BoxCutDesc()
    bc.n_bins, bc.lgs_lo, bc.lgs_hi, bc.cut_w, bc.cut_l, bc.e_a, bc.e_b, bc.mlp_cut = 4, 1.0, 5.0, 0.5, 0.5, -3.0, 1.0, 0.5
    for k in range(4):
        bc.w_mean[k], bc.w_std[k], bc.l_mean[k], bc.l_std[k] = 0.05, 0.02, 0.1, 0.05
    for f in range(10):
        bc.feat_lo[f], bc.feat_hi[f] = (1.5 if f == 0 else -100.0), (4.5 if f == 0 else 100.0)
    return m, bc


@pytest.mark.parametrize("n_evt", [1, 14, 511, 512, 513, 1500])
def test_event_pass_forms_agree(torch_dev, n_evt):
    import torch
    import dl0sim
    cams = [rta.Camera.from_type(c) for c in dl0sim.camera_types_c1()[:2]]
    pipe = rta.Pipeline(cams)
    m, bc = network()
    pipe.attach_mlp(m, bc)
    rec, ty, off, d_rec, d_ty, d_off = make(torch_dev, n_evt)
    say("event pass: %d events, %d telescopes" % (n_evt, len(ty)))
    whole = pipe.stereo(d_off, d_ty, d_rec.clone()).cpu()
    flags = d_rec.clone()
    pipe.stereo(d_off, d_ty, flags)
    parts = []
    for a in range(0, n_evt, 100):
        b = min(n_evt, a + 100)
        lo, hi = int(off[a]), int(off[b])
        parts.append(pipe.stereo((d_off[a:b + 1] - lo).contiguous(), d_ty[lo:hi].contiguous() if hi > lo else d_ty[:0],
                                 d_rec[lo:hi].clone()).cpu())
    assert torch.equal(whole.view(torch.int32), torch.cat(parts).view(torch.int32))
    cls = rta.classify(m, bc, d_rec).cpu().numpy().astype(np.float64)
    e = rta.records(whole, rta.EVENT_DTYPE)
    use = (ty >= 0) & ((rec["flags"] & rta.FLAG_HILLAS_INVALID) == 0)
    got = rta.records(flags)["flags"]
    assert np.array_equal((got & rta.FLAG_MLP_FALLBACK) != 0, use & (cls[:, 3] > 0))
    for k in range(n_evt):
        i = np.arange(off[k], off[k + 1])[use[off[k]:off[k + 1]]]
        assert int(e["n_tel"][k]) == off[k + 1] - off[k]
        if len(i) == 0:
            assert np.isnan(e["gammaness"][k]) and np.isnan(e["log10_energy"][k])
            continue
        w = rec["size"][i].astype(np.float64)
        for name, v in (("gammaness", cls[i, 0]), ("log10_energy", cls[i, 1])):
            # two sums of up to 130 float32 products and their quotient
            bound = (len(i) + 4) * 2.0 ** -23 * np.sum(w * np.abs(v)) / np.sum(w) * 2 + 1e-30
            assert abs(float(e[name][k]) - np.sum(w * v) / np.sum(w)) <= bound, (k, name)
    assert pipe.status() == 0


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32767, 32768, 32769, 65600])
def test_classify_rounds_agree(torch_dev, n):
    """rta_classify's persistent wavefronts: a record's outputs do not depend
    on the round or the row of the tile that it falls into."""
    import torch
    m, bc = network()
    d = make(torch_dev, 2400)[3]
    d = d[: n]
    assert d.shape[0] == n
    whole = rta.classify(m, bc, d)
    parts = torch.cat([rta.classify(m, bc, d[a:a + 1003].contiguous()) for a in range(0, n, 1003)])
    assert torch.equal(whole.view(torch.int32), parts.view(torch.int32))
    box = rta.classify(None, bc, d)
    assert bool((box[:, 3] == 1).all()) and torch.equal(box.view(torch.int32)[whole[:, 3] == 1],
                                                        whole.view(torch.int32)[whole[:, 3] == 1])
