"""The alert search at the edges of its tiles of whole grid rows: grids of one
cell, smaller than the reach, as wide as a workgroup, one row or several per
tile with a last tile that is not full, the longest reach, and a ring without
cells.  N_on / N_off, the alert set and the count are exact against sums of
shifted maps of the oracle's windows (compared with the oracle's own loops on
the small grids, which take a minute on the large ones); the FP64 significance agrees to rounding
(two logarithms and a root of sums of counts: 1e-12)."""
import numpy as np
import pytest

import paper_1307_6489_amd as rta
from oracle import sam as osam

pytestmark = pytest.mark.gpu


def shifted_search(C, end_bin, p):
    G = p["grid"]
    on2, in2, out2 = osam.f32(p["r_on"]) ** 2, osam.f32(p["r_in"]) ** 2, osam.f32(p["r_out"]) ** 2
    R = int(np.ceil(osam.f32(p["r_out"])))
    out, alerts = [], []
    for s, w in enumerate(p["scales"]):
        maps = np.stack([osam.window(C, end_bin, w), np.ones((G, G), np.int64)])
        pad = np.pad(maps, ((0, 0), (R, R), (R, R)))
        on, off = np.zeros_like(maps), np.zeros_like(maps)
        for dy in range(-R, R + 1):
            for dx in range(-R, R + 1):
                part = pad[:, R + dy:R + dy + G, R + dx:R + dx + G]
                if dx * dx + dy * dy <= on2:
                    on += part
                elif in2 < dx * dx + dy * dy <= out2:
                    off += part
        S = np.array([osam.li_ma_cells(*map(int, v)) for v in
                      zip(on[0].ravel(), off[0].ravel(), on[1].ravel(), off[1].ravel())]).reshape(G, G)
        out.append({"S": S, "N_on": on[0], "N_off": off[0]})
        alerts += [(s, int(x), int(y), S[y, x]) for y, x in np.argwhere(S >= p["sigma_alert"])]
    return out, alerts


@pytest.mark.parametrize("grid,r_on,r_in,r_out", [
    (1, 0.0, 0.3, 0.6), (1, 1.0, 2.0, 3.0), (3, 1.0, 2.0, 16.0), (16, 1.5, 3.5, 7.0), (17, 0.0, 1.0, 2.3),
    (50, 2.0, 2.5, 9.9), (100, 1.5, 3.5, 7.0), (129, 3.0, 10.0, 16.0), (255, 1.0, 1.5, 2.0), (256, 1.5, 14.5, 16.0)])
def test_search_over_tiles(grid, r_on, r_in, r_out):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = {"grid": grid, "cell": 0.0015, "t0": 0.0, "bin_s": 1.0, "n_bins": 67, "r_on": r_on, "r_in": r_in,
         "r_out": r_out, "gamma_cut": 0.5, "scales": [1, 5, 67], "sigma_alert": 2.5}
    print("alert search over tiles: grid", grid, flush=True)
    rng = np.random.default_rng(grid)
    n = 4000
    rec = np.zeros(n, rta.EVENT_DTYPE)
    half = 0.55 * grid * p["cell"]
    rec["dir_x"] = rng.uniform(-half, half, n)
    rec["dir_y"] = rng.uniform(-half, half, n)
    rec["gammaness"] = rng.uniform(0.4, 1.0, n)
    t = rng.uniform(-1.0, 68.0, n)
    d = np.stack([rec["dir_x"], rec["dir_y"]], 1)
    C, used = osam.histogram(d, t, rec["gammaness"], np.ones(n, bool), p)
    sam = rta.Sam(grid, p["n_bins"], p["t0"], p["bin_s"], p["cell"], r_on, r_in, r_out, p["gamma_cut"],
                  p["sigma_alert"], p["scales"])
    sam.fill(torch.from_numpy(rec.view(np.float32).reshape(-1, 8).copy()).cuda(), torch.from_numpy(t).cuda())
    assert np.array_equal(sam.counts().astype(np.int64), C) and used > 0
    for end_bin in (0, 66):
        ref, ref_alerts = shifted_search(C, end_bin, p)
        if grid <= 17:
            loops, loop_alerts = osam.search(C, end_bin, p)
            assert all(np.array_equal(a[k], b[k]) for a, b in zip(ref, loops) for k in ("S", "N_on", "N_off"))
            assert [a[:3] for a in ref_alerts] == [a[:3] for a in loop_alerts]
        sig, non, noff, alerts, found = sam.search(end_bin, max_alerts=3 * grid * grid)
        for s, r in enumerate(ref):
            assert np.array_equal(non[s].cpu().numpy(), r["N_on"])
            assert np.array_equal(noff[s].cpu().numpy(), r["N_off"])
            assert np.allclose(sig[s].cpu().numpy(), r["S"], rtol=1e-12, atol=1e-12)
        near = {(s, x, y) for s, x, y, v in ref_alerts if abs(v - p["sigma_alert"]) < 1e-9}
        got = {(int(a["scale"]), int(a["ix"]), int(a["iy"])) for a in alerts}
        assert len(got) == len(alerts) == found
        assert got - near == {(s, x, y) for s, x, y, v in ref_alerts} - near
        assert sam.search(end_bin, max_alerts=0, maps=False)[4] == found
    sam.clear()
    assert not sam.counts().any()
