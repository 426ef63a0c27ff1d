"""The calibration's outputs are stored in runs of consecutive pixels: odd and
even cameras of one pixel to more than a workgroup's, several events (an odd
camera's later events begin at any address), byte outputs at odd addresses,
single outputs alone, and nothing written before or after an output.  Values
as the oracle's: integers exact, q and t to the rounding of a float division
(1e-6)."""
import ctypes

import numpy as np
import pytest

import dl0sim
import oracle
import paper_1307_6489_amd as rta

pytestmark = pytest.mark.gpu
SIZE = {"S": 4, "D": 4, "sstar": 1, "peak": 1, "gain": 1, "q": 4, "t": 4}
TYPE = {"S": np.int32, "D": np.int32, "sstar": np.uint8, "peak": np.uint8, "gain": np.uint8, "q": np.float32,
        "t": np.float32}


@pytest.mark.parametrize("n_pix,n_gain", [(1, 2), (2, 1), (3, 2), (65, 1), (511, 2), (512, 2), (513, 2), (1855, 1)])
def test_runs(n_pix, n_gain):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("calibration runs:", n_pix, n_gain, flush=True)
    ct = dl0sim.CameraType("runs", n_pix, 20, n_gain, 10.0)
    rng = np.random.default_rng(n_pix)
    E = 5
    tr = rng.integers(250, 400, size=(E, n_gain, 20, ct.n_pix_pad), dtype=np.uint16)
    if n_gain == 2:
        tr[:, 0, 7, ::3] = 4095        # switched pixels
    ref = oracle.calibrate_events(oracle.Camera.from_type(ct), tr)
    cam = rta.Camera.from_type(ct)
    dev = torch.from_numpy(tr).cuda()
    for want in (list(SIZE), ["D", "gain"], ["t"]):
        buf = {k: torch.full((64 + E * n_pix * SIZE[k] + 64,), 0xA5, dtype=torch.uint8, device="cuda") for k in want}
        lead = {k: 60 if SIZE[k] == 4 else 61 for k in want}
        p = [ctypes.c_void_p(buf[k].data_ptr() + lead[k]) if k in want else None for k in SIZE]
        rta._check(rta.lib().rta_calibrate(cam.handle, ctypes.c_void_p(dev.data_ptr()), E, *p, None))
        torch.cuda.synchronize()
        for k in want:
            b = buf[k].cpu().numpy()
            end = lead[k] + E * n_pix * SIZE[k]
            assert (b[:lead[k]] == 0xA5).all() and (b[end:] == 0xA5).all(), k
            v = np.frombuffer(b[lead[k]:end].tobytes(), TYPE[k]).reshape(E, n_pix)
            if k in ("q", "t"):
                assert np.allclose(v, ref[k], rtol=1e-6, atol=1e-6 if k == "q" else 1e-5), k
            else:
                assert np.array_equal(v.astype(np.int64), ref[k].astype(np.int64)), k
