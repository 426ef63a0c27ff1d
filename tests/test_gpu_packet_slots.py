"""The packet decode with one, two and four slots of lanes per packet: packet
counts on either side of the two counts where the slots change and a mean
packet size above the line, cameras whose sample rows number fewer than a
block, a block, and not a multiple of blocks and slots (4 to 66 rows), rows of
2 bytes up to the longest.  Some packets have one bit changed in the first or
the last sample row.  Pool, records, CRCs and types are exact against the
oracle."""
import numpy as np
import pytest

import dl0sim
import dl0sim.workloads as W
import paper_1307_6489_amd as rta
from dl0sim import packets as gp
from oracle import packets as op

pytestmark = pytest.mark.gpu

SMALL = [(1, 4, 1), (37, 5, 1), (8, 7, 2), (9, 33, 2)]
WIDE = [(2047, 11, 1), (2048, 16, 2), (520, 33, 1), (513, 8, 1)]


@pytest.mark.parametrize("shapes,n", [(SMALL, 1), (SMALL, 40), (SMALL, 300), (SMALL, 600), (WIDE, 12), (WIDE, 257),
                                      (WIDE, 513), ([(1855, 25, 1)], 520)])
def test_slots(shapes, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("packet slots: %d packets of %s" % (n, shapes), flush=True)
    rng = np.random.default_rng(n)
    cts = [dl0sim.CameraType("p%d" % k, N, T, G, 10.0) for k, (N, T, G) in enumerate(shapes)]
    types = rng.integers(0, len(cts), n).astype(np.int32)
    elems = np.array([c.event_elems for c in cts], np.int64)[types]
    blob = rng.integers(0, 65536, int(elems.sum()), dtype=np.uint16)
    pool = W.Pool(cts, blob, types, np.concatenate([[0], np.cumsum(elems)[:-1]]), None)
    st, off = gp.serialize(pool, np.arange(n), seed=3)
    bad = np.arange(2, n, 5)
    for k in bad:
        row = 2 * cts[types[k]].n_pix
        at = 32 + (0 if k % 2 else 2 * cts[types[k]].n_gain * cts[types[k]].n_samp * cts[types[k]].n_pix - row)
        st[off[k] + at + rng.integers(0, row)] ^= 1 << rng.integers(0, 8)
    cams = [rta.Camera.from_type(c) for c in cts]
    pipe = rta.Pipeline(cams, do_stereo=False)
    o, t, po, size, used = rta.frame_packets(cams, st)
    dev = torch.device("cuda:0")
    t_dev = torch.from_numpy(t.copy()).to(dev)
    data, nb = rta.packet_buffer(st, dev)
    pool_d, rec = rta.decode_packets(pipe, data, torch.from_numpy(o).to(dev), t_dev, torch.from_numpy(po).to(dev),
                                     size, n_bytes=nb)
    torch.cuda.synchronize()
    ref_pool, ref_rec, ref_t = op.decode(st, o, t, po, size, shapes)
    got = rec.cpu().numpy().view(rta.PACKET_DTYPE).reshape(-1)
    for f in ("event_number", "cam_type", "flags", "crc_stored", "crc_computed"):
        assert np.array_equal(got[f], ref_rec[f]), f
    assert np.array_equal(np.flatnonzero(ref_rec["flags"]), bad)
    assert np.array_equal(t_dev.cpu().numpy(), ref_t)
    assert np.array_equal(pool_d.cpu().numpy()[:size], ref_pool)
