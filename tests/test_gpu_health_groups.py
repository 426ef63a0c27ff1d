"""The health monitor at the edges of its groups of 8 samples and of its
median by radix passes.  Everything is exact: the sums are integers, mean and
rms are the same FP64 expressions without contraction, the median is one of
the values.

Traces shorter than, as long as and longer than a group, with 16-bit samples
up to 65535; a switch level of zero (every sample counts as saturated); more
events than slots and fewer; medians among equal values, two values, values
of one binary exponent and of many, with one, 64, 65 and 2048 pixels; sums
beyond what 32 bits of byte products hold."""
import numpy as np
import pytest

import dl0sim
import paper_1307_6489_amd as rta
from oracle import health as oh

pytestmark = pytest.mark.gpu
P = {"rms_dead": 0.5, "noisy_factor": 1.5, "ped_tol": 20.0, "sat_frac": 0.01, "bad_frac_max": 0.05}


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rta.lib()
    return torch.device("cuda:0")


def check(ct, tr, dev):
    import torch
    pix, c = rta.health(rta.Camera.from_type(ct), torch.from_numpy(np.ascontiguousarray(tr)).to(dev), **P)
    rp, rc = oh.health(tr, ct.n_pix, ct.n_gain, ct.ped, ct.hg_switch_adc, P)
    for k in ("S1", "S2", "n_sat"):
        assert np.array_equal(pix[k.lower()].astype(np.int64), rp[k]), k
    assert np.array_equal(pix["mean"], rp["mean"]) and np.array_equal(pix["rms"], rp["rms"])
    assert np.array_equal(pix["flags"].astype(np.int64), rp["flags"])
    assert np.array_equal(c["median_rms"][:ct.n_gain], rc["median_rms"])
    assert int(c["n_bad"]) == rc["n_bad"] and int(c["verdict"]) == rc["verdict"]


@pytest.mark.parametrize("n_samp,n_gain,n_evt,level", [(8, 2, 3, 0), (9, 2, 1, 4000), (15, 1, 70, 4000),
                                                       (16, 2, 600, 65535), (33, 2, 150, 30000)])
def test_groups(torch_dev, n_samp, n_gain, n_evt, level):
    ct = dl0sim.CameraType("groups", 37, n_samp, n_gain, 10.0)
    ct.hg_switch_adc = level
    rng = np.random.default_rng(n_samp + n_evt)
    tr = rng.integers(0, 65536, size=(n_evt, n_gain, n_samp, 40), dtype=np.uint16)
    tr[:, :, :, ::3] //= 16
    tr[0, 0, n_samp - 1, 5] = 65535
    print("health groups:", n_samp, n_gain, n_evt, flush=True)
    check(ct, tr, torch_dev)


@pytest.mark.parametrize("n_pix", [1, 2, 64, 65, 130, 2048])
@pytest.mark.parametrize("kind", ["equal", "two", "close", "wide"])
def test_medians(torch_dev, n_pix, kind):
    ct = dl0sim.CameraType("medians", n_pix, 32, 2, 10.0)
    rng = np.random.default_rng(n_pix)
    npad = (n_pix + 7) // 8 * 8
    amp = {"equal": np.full((2, npad), 7), "two": rng.integers(3, 5, (2, npad)),
           "close": rng.integers(1000, 1020, (2, npad)), "wide": 2 ** rng.integers(0, 14, (2, npad))}[kind]
    if kind == "equal":
        amp[1] = 0
    tr = np.full((2, 2, 32, npad), 20000, np.uint16)
    tr[:, :, ::2] += amp[None, :, None].astype(np.uint16)
    if kind == "close":          # rms that differ in their last bits only
        tr[:, :, 5] += rng.integers(0, 3, (2, 2, npad)).astype(np.uint16)
    print("health medians:", n_pix, kind, flush=True)
    check(ct, tr, torch_dev)


def test_sums_beyond_32_bits(torch_dev):
    """264000 events of 255 samples of one pixel, nearly all 65535: a slot
    takes more groups than its 32-bit sums of byte products hold."""
    import torch
    E, T = 264000, 255
    ct = dl0sim.CameraType("long", 1, T, 1, 10.0)
    tr = torch.full((E, T, 8), -1, dtype=torch.int16, device=torch_dev)      # 65535 in 16 bits
    tr[::1000, ::7, 0] = 12345
    tr[-1, -1, 0] = 3
    print("health: %d events of one pixel" % E, flush=True)
    pix, c = rta.health(rta.Camera.from_type(ct), tr.view(torch.uint16).reshape(-1), **P)
    n_mid = len(range(0, E, 1000)) * len(range(0, T, 7))
    full = E * T - n_mid - 1
    assert int(pix["s1"][0][0]) == full * 65535 + n_mid * 12345 + 3
    assert int(pix["s2"][0][0]) == full * 65535 ** 2 + n_mid * 12345 ** 2 + 9
    assert int(pix["n_sat"][0][0]) == full
