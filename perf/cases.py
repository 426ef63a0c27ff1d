"""Timed cases of the reconstruction library, through its public entry points.

Each case is one piece of work that a program built on the library has it do:

  reconstruct   Pipeline.process over a batch of camera events (calibration,
                cleaning, image parameters, and per array event the stereo
                direction, with or without the gamma/hadron network)
  stages        calibrate -> clean -> hillas with the per-pixel products kept
  packets       decode_packets over a device-resident telemetry stream
  health        health over a batch of pedestal events
  alerts        Sam.clear, Sam.fill and Sam.search over an event list
  train         Adam steps of the network on rows of a training set
  classify      network + box-cut decisions of image-parameter records

Inputs are made on the GPU from the seed alone: hexagonal cameras with a
per-pixel spread of pedestals and gains, traces of one Cherenkov ellipse per
camera event over night-sky and electronic noise, 1 ns samples, sizes from
50 to 20000 photo-electrons (the brightest switch pixels to the low gain).
The layout of a batch (camera types, multiplicities) belongs to the case; the
values belong to the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1307_6489_amd as rta

DEV = "cuda"
WINDOW = 4
SWITCH_ADC = 4000
T_PIC, T_BND = 10.0, 5.0
PITCH = 0.05
ADC_PER_PE = (10.0, 0.625)
NSB = 0.1          # photo-electrons per sample
EXTRACTORS = {"sliding": 0, "fixed": 1, "global": 2, "neighbour": 3}
# pixels x samples x gains * weight, of the throughput mix
MIX = "1855x40x2*1,1764x25x2*3,2048x128x2*6"
# the same three cameras as the paced array events hold them
MIX_ARRAY = "1855x40x2*1,1764x25x2*1,2048x128x2*8"
FOCAL = {1855: 28.0, 1764: 16.0, 2048: 5.6}
SCALES = (1, 10, 60, 600, 3600)
# bytes of high-gain trace that a drawn batch may hold (the largest listed one has about this)
MOST_TRACE_BYTES = 5.6e9


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one array event as it arrives (the event-by-event analysis of the paced stream): latency counts
        {"name": "array_event", "op": "reconstruct", "cameras": MIX_ARRAY, "array_events": 1, "mult_lo": 21,
         "mult_hi": 21, "extractor": "sliding", "classify": "camera"},
        # a few seconds' worth of array events with the network in the event pass
        {"name": "array_events_100", "op": "reconstruct", "cameras": MIX, "array_events": 100, "mult_lo": 2,
         "mult_hi": 40, "extractor": "sliding", "classify": "event"},
        # bulk reprocessing of camera events with the default extractor: the headline path
        {"name": "mix_sliding", "op": "reconstruct", "cameras": MIX, "telescopes": 16000, "extractor": "sliding",
         "classify": "none"},
        # the same with the other signal extractors
        {"name": "mix_fixed", "op": "reconstruct", "cameras": MIX, "telescopes": 8000, "extractor": "fixed",
         "classify": "none"},
        {"name": "mix_global", "op": "reconstruct", "cameras": MIX, "telescopes": 8000, "extractor": "global",
         "classify": "none"},
        {"name": "mix_neighbour", "op": "reconstruct", "cameras": MIX, "telescopes": 8000, "extractor": "neighbour",
         "classify": "none"},
        # per-pixel products wanted: the single-gain 1855 x 30 camera through the unfused calls
        {"name": "stages_1855x30", "op": "stages", "cameras": "1855x30x1*1", "events": 1000},
        # a received chunk of the telemetry stream turned into a trace pool
        {"name": "packets_mix", "op": "packets", "cameras": MIX, "packets": 2000},
        # the data-quality check of one camera's pedestal events
        {"name": "health_2048x128", "op": "health", "cameras": "2048x128x2*1", "events": 500},
        # an event list scanned for transients on five timescales
        {"name": "alerts_64", "op": "alerts", "grid": 64, "events": 1080000},
        # network training on rows of a training set
        {"name": "train_4096", "op": "train", "batch": 4096, "steps": 20, "rows": 200000},
        # classification of a run's records
        {"name": "classify_200k", "op": "classify", "records": 200000},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_camera(rng):
    # single and dual gain, full and partial last pixel groups, traces from a few samples to the longest
    n_pix = rng.choice([1855, 1764, 2048, _log_int(rng, 61, 2048), _log_int(rng, 397, 2048)])
    n_samp = rng.choice([25, 30, 40, 128, _log_int(rng, 8, 255)])
    return "%dx%dx%d*1" % (n_pix, n_samp, rng.choice([1, 2, 2]))


def draw(rng):
    op = rng.choice(["reconstruct"] * 6 + ["stages", "stages", "packets", "health", "alerts", "train", "classify"])
    if op == "reconstruct":
        cams = rng.choice([MIX, MIX_ARRAY, _draw_camera(rng)])
        c = {"op": op, "cameras": cams, "extractor": rng.choice(["sliding", "sliding"] + list(EXTRACTORS)),
             "classify": rng.choice(["none", "none", "camera", "event"])}
        most = int(min(16000, MOST_TRACE_BYTES / _mean_trace_bytes(cams)))
        if rng.random() < 0.5:
            lo = rng.randint(2, 10)
            hi = rng.randint(lo, 40)
            c.update(array_events=_log_int(rng, 1, max(1, most // 40)), mult_lo=lo, mult_hi=hi)
        else:
            c["telescopes"] = _log_int(rng, 1, most)
            if c["classify"] == "event":
                c["classify"] = "camera"
        return c
    if op in ("stages", "health"):
        cams = _draw_camera(rng)
        cap = (2.0e9 if op == "stages" else 1.0e9) / _mean_trace_bytes(cams)
        return {"op": op, "cameras": cams, "events": _log_int(rng, 1, max(1, min(4000, int(cap))))}
    if op == "packets":
        cams = rng.choice([MIX, _draw_camera(rng)])
        return {"op": op, "cameras": cams,
                "packets": _log_int(rng, 1, max(1, min(4000, int(0.7e9 / _mean_trace_bytes(cams)))))}
    if op == "alerts":
        return {"op": op, "grid": rng.randint(16, 128), "events": _log_int(rng, 1000, 10800000)}
    if op == "train":
        return {"op": op, "batch": _log_int(rng, 100, 16384), "steps": rng.randint(1, 20), "rows": 200000}
    return {"op": "classify", "records": _log_int(rng, 16, 2000000)}


# ---------------------------------------------------------------------------
# Cameras
# ---------------------------------------------------------------------------
class _Camera:
    """Tables of one camera type: host arrays as a program reads them from its
    configuration, device copies for making the traces."""

    def __init__(self, n_pix, n_samp, n_gain):
        self.n_pix, self.n_samp, self.n_gain = n_pix, n_samp, n_gain
        self.n_pad = (n_pix + 7) // 8 * 8
        self.focal = FOCAL.get(n_pix, 16.0)
        self.elems = n_gain * n_samp * self.n_pad
        self.x, self.y, self.nbr = _hexagon(n_pix)
        r = np.random.default_rng(n_pix)
        spread = 1.0 + 0.05 * (2.0 * r.random(n_pix) - 1.0)
        base = 300.0 + 5.0 * (2.0 * r.random((2, n_pix)) - 1.0)
        gain = np.array(ADC_PER_PE)[:, None] * spread
        self.adc = np.ascontiguousarray(gain[:n_gain].astype(np.float32))
        self.base = np.ascontiguousarray(base[:n_gain].astype(np.float32))
        # the pedestal per sample holds the mean night-sky background
        self.ped = (self.base.astype(np.float64) + self.adc.astype(np.float64) * NSB).astype(np.float32)
        self.radius = float(np.sqrt(self.x.astype(np.float64) ** 2 + self.y.astype(np.float64) ** 2).max())

    def handle(self):
        return rta.Camera(self.n_pix, self.n_samp, self.n_gain, self.x, self.y, self.nbr, self.ped, self.adc,
                          self.focal, WINDOW, SWITCH_ADC, T_PIC, T_BND)


@functools.lru_cache(maxsize=64)
def _hexagon(n_pix):
    """The n_pix points of a hexagonal lattice nearest the centre, ordered by
    distance and angle, and the six neighbours of each (-1: none)."""
    m = int(math.sqrt(n_pix)) + 3
    a, b = np.meshgrid(np.arange(-m, m + 1), np.arange(-m, m + 1), indexing="ij")
    a, b = a.ravel(), b.ravel()
    x, y = PITCH * (a + 0.5 * b), PITCH * math.sqrt(0.75) * b
    order = np.lexsort((np.arctan2(y, x), a * a + a * b + b * b))[:n_pix]
    a, b = a[order], b[order]
    at = np.full((2 * m + 5, 2 * m + 5), -1, np.int32)
    at[a + m + 2, b + m + 2] = np.arange(n_pix)
    step = [(1, 0), (0, 1), (-1, 1), (-1, 0), (0, -1), (1, -1)]
    nbr = np.stack([at[a + da + m + 2, b + db + m + 2] for da, db in step], 1).astype(np.int32)
    return x[order].astype(np.float32), y[order].astype(np.float32), np.ascontiguousarray(nbr)


@functools.lru_cache(maxsize=64)
def _camera(n_pix, n_samp, n_gain):
    return _Camera(n_pix, n_samp, n_gain)


def _cameras(text):
    cams, weights = [], []
    for part in text.split(","):
        dims, w = part.split("*")
        cams.append(_camera(*(int(v) for v in dims.split("x"))))
        weights.append(float(w))
    return cams, np.array(weights) / sum(weights)


def _mean_trace_bytes(text):
    """High-gain trace bytes of a camera event, over the types."""
    total, weight = 0.0, 0.0
    for part in text.split(","):
        dims, w = part.split("*")
        n, t, _ = (int(v) for v in dims.split("x"))
        total += float(w) * n * t * 2
        weight += float(w)
    return total / weight


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _layout(case):
    """Camera type of every camera event, and the array events' ranges (None
    without array events): part of the case, not of the seed."""
    cams, w = _cameras(case["cameras"])
    r = np.random.default_rng(20130724)
    if case.get("array_events"):
        mult = r.integers(case["mult_lo"], case["mult_hi"] + 1, case["array_events"])
        off = np.zeros(len(mult) + 1, np.int64)
        off[1:] = np.cumsum(mult)
        return r.choice(len(cams), int(off[-1]), p=w).astype(np.int32), off
    n = case.get("telescopes") or case.get("events") or case.get("packets")
    counts = np.floor(w * n).astype(np.int64)
    for i in np.argsort(-(w * n - counts), kind="stable")[: n - counts.sum()]:
        counts[i] += 1
    types = np.repeat(np.arange(len(cams), dtype=np.int32), counts)
    r.shuffle(types)
    return types, None


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, lo, hi):
    return lo + (hi - lo) * torch.rand(n, generator=g, device=DEV)


def _images(cam, n, g, src=None, signal=True):
    """Image parameters of n camera events; with src (nominal frame) the major
    axes point at the source."""
    rmax = min(0.8, 0.8 * cam.radius)
    r, ph = rmax * torch.sqrt(_uniform(g, n, 0, 1)), _uniform(g, n, 0, 2 * math.pi)
    cx, cy = r * torch.cos(ph), r * torch.sin(ph)
    width = _uniform(g, n, 0.02, 0.06)
    size = torch.exp(_uniform(g, n, math.log(50.0), math.log(20000.0))) * (1.0 if signal else 0.0)
    psi = _uniform(g, n, -math.pi / 2, math.pi / 2)
    if src is not None:
        psi = torch.atan2(src[:, 1] - cy / cam.focal, src[:, 0] - cx / cam.focal)
    return dict(cx=cx, cy=cy, w=width, len=width * _uniform(g, n, 1.5, 4.0), size=size, psi=psi,
                t0=cam.n_samp / 2.0 + _uniform(g, n, -2.0, 2.0), grad=_uniform(g, n, -5.0, 5.0))


def _render(cam, im, g, out):
    """Traces uint16 [n][G][T][Npad] of the images into out (its int16 view)."""
    n_all = len(im["size"])
    x, y = torch.from_numpy(cam.x).to(DEV), torch.from_numpy(cam.y).to(DEV)
    area = math.sqrt(0.75) * PITCH * PITCH
    step = max(1, int(48e6 / (cam.n_samp * cam.n_pad)))
    k = torch.arange(cam.n_samp, device=DEV, dtype=torch.float32)
    for a in range(0, n_all, step):
        s = {key: v[a:a + step, None] for key, v in im.items()}
        n = len(s["size"])
        dx, dy = x[None] - s["cx"], y[None] - s["cy"]
        lon = dx * torch.cos(s["psi"]) + dy * torch.sin(s["psi"])
        tra = dy * torch.cos(s["psi"]) - dx * torch.sin(s["psi"])
        mean = s["size"] * area / (2 * math.pi * s["len"] * s["w"]) * torch.exp(
            -0.5 * ((lon / s["len"]) ** 2 + (tra / s["w"]) ** 2))
        npe = torch.poisson(mean, generator=g)
        # Gaussian pulse of 2 ns, unit area
        pulse = torch.exp(-0.125 * (k[None, :, None] - (s["t0"] + s["grad"] * lon)[:, None, :]) ** 2)
        pulse *= (npe / (2.0 * math.sqrt(2 * math.pi)))[:, None, :]
        for gain in range(cam.n_gain):
            adc = torch.from_numpy(cam.adc[gain]).to(DEV)
            v = torch.randn((n, cam.n_samp, cam.n_pix), generator=g, device=DEV)
            v *= torch.sqrt(25.0 + NSB * adc * adc)
            v += torch.from_numpy(cam.ped[gain]).to(DEV)
            v.addcmul_(pulse, adc[None, None, :].expand_as(pulse))
            v.round_().clamp_(0, 4095 if cam.n_gain == 2 and gain == 0 else 65535)
            out[a:a + n, gain, :, :cam.n_pix] = v.to(torch.int32).to(torch.int16)


def _traces(case, seed, signal=True):
    """(cams, types, event ranges, pool int16, element offset of every camera
    event, per type its camera events' indices and traces)."""
    cams, _ = _cameras(case["cameras"])
    types, ev_off = _layout(case)
    g = _gen(seed)
    src = None
    if ev_off is not None:
        n_ev = len(ev_off) - 1
        r, ph = 0.02 * torch.sqrt(_uniform(g, n_ev, 0, 1)), _uniform(g, n_ev, 0, 2 * math.pi)
        mult = torch.from_numpy(np.diff(ev_off)).to(DEV)
        src = torch.repeat_interleave(torch.stack([r * torch.cos(ph), r * torch.sin(ph)], 1), mult, dim=0)
    idx = [np.nonzero(types == t)[0] for t in range(len(cams))]
    start = np.cumsum([0] + [len(i) * c.elems for i, c in zip(idx, cams)])
    pool = torch.zeros(max(int(start[-1]), 8), dtype=torch.int16, device=DEV)
    off = np.zeros(len(types), np.int64)
    groups = []
    for t, cam in enumerate(cams):
        n = len(idx[t])
        off[idx[t]] = start[t] + np.arange(n) * cam.elems
        if n == 0:
            groups.append((idx[t], None))
            continue
        view = pool[int(start[t]):int(start[t + 1])].view(n, cam.n_gain, cam.n_samp, cam.n_pad)
        im = _images(cam, n, g, None if src is None else src[torch.from_numpy(idx[t]).to(DEV)], signal)
        _render(cam, im, g, view)
        groups.append((idx[t], view))
    return cams, types, ev_off, pool, off, groups


# Mean and spread of the network's inputs, the range it was trained on, and
# box cuts, of the kind that a trained configuration holds.
FEAT_MEAN = np.array([2.9, 0.085, 0.045, 0.5, 0.0, 0.0, 2.4, 0.0, 0.05, 1.05], np.float32)
FEAT_STD = np.array([0.7, 0.04, 0.02, 0.25, 0.9, 0.35, 0.5, 4.0, 0.15, 0.3], np.float32)
FEAT_LO = np.array([1.5, 0.01, 0.0, 0.0, -1.58, -1.5, 1.0, -30.0, 0.0, 1.0], np.float32)
FEAT_HI = np.array([4.6, 0.3, 0.12, 1.3, 1.58, 1.5, 6.0, 30.0, 0.9, 4.0], np.float32)


def _network(seed):
    """Packed parameters, as a training leaves them in size."""
    r = np.random.default_rng([7, int(seed)])
    parts = []
    for n_in, n_out in ((10, 64), (64, 64), (64, 64), (64, 2)):
        parts.append(r.standard_normal((n_in, n_out)) * math.sqrt(2.0 / n_in))
        parts.append(0.1 * r.standard_normal(n_out))
    return np.concatenate([p.ravel() for p in parts]).astype(np.float32)


def _boxcut():
    bc = rta.BoxCutDesc()
    bc.n_bins, bc.lgs_lo, bc.lgs_hi = 20, 1.5, 4.6
    for k in range(20):
        bc.w_mean[k], bc.w_std[k] = 0.035 + 0.0005 * k, 0.012
        bc.l_mean[k], bc.l_std[k] = 0.07 + 0.001 * k, 0.03
    bc.cut_w, bc.cut_l, bc.e_a, bc.e_b, bc.mlp_cut = 0.9, 1.4, -3.0, 1.0, 0.5
    for f in range(10):
        bc.feat_lo[f], bc.feat_hi[f] = float(FEAT_LO[f]), float(FEAT_HI[f])
    return bc


def _mlp(seed, max_batch=4096):
    m = rta.Mlp(max_batch=max_batch)
    m.set_params(_network(seed), FEAT_MEAN, FEAT_STD)
    return m


def _sky(case, seed):
    """An hour's event list: background over the field, a gamma-like tenth,
    and one flare in the last minute.  Event records [n][8] and times."""
    g, n = _gen(seed), case["events"]
    n_src = n // 100
    t = _uniform(g, n, 0, 3600.0).double()
    r, ph = 0.05 * torch.sqrt(_uniform(g, n, 0, 1)), _uniform(g, n, 0, 2 * math.pi)
    x, y = r * torch.cos(ph), r * torch.sin(ph)
    score = _uniform(g, n, 0, 0.5)
    hot = _uniform(g, n, 0, 1) < 0.1
    score[hot] = _uniform(g, n, 0.7, 1.0)[hot]
    t[:n_src] = 3540.0 + 60.0 * torch.rand(n_src, generator=g, device=DEV).double()
    x[:n_src] = 0.010 + 0.0008 * torch.randn(n_src, generator=g, device=DEV)
    y[:n_src] = 0.004 + 0.0008 * torch.randn(n_src, generator=g, device=DEV)
    score[:n_src] = _uniform(g, n_src, 0.75, 1.0)
    t, order = torch.sort(t)
    e = torch.zeros((n, 8), dtype=torch.float32, device=DEV)
    e[:, 0], e[:, 1], e[:, 3] = x[order], y[order], score[order]
    bad = _uniform(g, n, 0, 1) < 0.02
    e.view(torch.int32)[:, 7] = bad.to(torch.int32) * rta.EVT_STEREO_INVALID
    return e, t


def _image_records(n, seed):
    """n image-parameter records [n][16] with the spread of a run's images."""
    g = _gen(seed)
    rec = torch.zeros((n, 16), dtype=torch.float32, device=DEV)
    mean, std = torch.from_numpy(FEAT_MEAN).to(DEV), torch.from_numpy(FEAT_STD).to(DEV)
    f = mean + std * torch.randn((n, 10), generator=g, device=DEV).clamp_(-2.2, 2.2)
    rec[:, 0] = 10.0 ** f[:, 0]
    rec[:, 3], rec[:, 4] = f[:, 1].abs(), f[:, 2].abs()
    rec[:, 11] = f[:, 3].abs()
    rec[:, 5] = f[:, 4].clamp(-1.57, 1.57)
    rec[:, 6], rec[:, 7], rec[:, 8] = f[:, 5], f[:, 6], f[:, 7]
    rec[:, 10] = f[:, 8].clamp(0.0, 1.0)
    rec.view(torch.int32)[:, 13] = f[:, 9].round().clamp_(1, 4).to(torch.int32)
    rec.view(torch.int32)[:, 12] = 30
    return rec


def _training_set(case, seed):
    g, n = _gen(seed), case["rows"]
    mean, std = torch.from_numpy(FEAT_MEAN).to(DEV), torch.from_numpy(FEAT_STD).to(DEV)
    z = torch.randn((n, 10), generator=g, device=DEV)
    label = ((z[:, 1] - z[:, 2] + 0.5 * z[:, 5] + 0.7 * torch.randn(n, generator=g, device=DEV)) > 0).float()
    log10e = z[:, 0] + 0.1 * torch.randn(n, generator=g, device=DEV)
    rows = torch.randint(0, n, (case["steps"], case["batch"]), generator=g, device=DEV)
    return (mean + std * z).contiguous(), label, log10e, [rows[i].contiguous() for i in range(case["steps"])]


# --- the packet stream: words of 16 bits, CRC-16 by pairwise combination ----
def _times_x(v, n):
    for _ in range(n):
        v = v << 1
        v = np.where(v & 0x10000, v ^ 0x11021, v)
    return v


@functools.lru_cache(maxsize=1)
def _crc_tables():
    """tables[k][v] = v x^(16 2^k) modulo the CRC polynomial."""
    tables = [_times_x(np.arange(65536), 16)]
    for _ in range(20):
        tables.append(tables[-1][tables[-1]])
    return [torch.from_numpy(t.astype(np.int32)).to(DEV) for t in tables]


def _crc16(words):
    """CRC-16 (register 0xFFFF) of the rows of words, int32 [n][m]."""
    tables = _crc_tables()
    words = words.clone()
    words[:, 0] ^= 0xFFFF
    v = tables[0][words.long()]
    k = 0
    while v.shape[1] > 1:
        if v.shape[1] & 1:  # leading zeros do not change the remainder
            v = torch.cat([torch.zeros_like(v[:, :1]), v], 1)
        v = tables[k][v[:, 0::2].long()] ^ v[:, 1::2]
        k += 1
    return v[:, 0]


def _stream(case, seed):
    """The packets of a mix in order of arrival: bytes on the device, packet
    offsets, types, pool offsets, pool size."""
    cams, types, _, _, _, groups = _traces(case, seed)
    size = np.array([34 + 2 * c.n_gain * c.n_samp * c.n_pix for c in cams], np.int64)[types]
    off = np.concatenate([[0], np.cumsum(size)])
    elems = np.array([c.elems for c in cams], np.int64)[types]
    slot = np.concatenate([[0], np.cumsum(elems)])
    buf = torch.zeros((int(off[-1]) + rta.PACKET_PAD + 1) // 2, dtype=torch.int16, device=DEV)
    for t, cam in enumerate(cams):
        idx, view = groups[t]
        for a in range(0, len(idx), 128):
            part = idx[a:a + 128]
            n = len(part)
            w = torch.zeros((n, 16), dtype=torch.int32, device=DEV)
            no = torch.from_numpy(part.astype(np.int32)).to(DEV)
            total = 34 + 2 * cam.n_gain * cam.n_samp * cam.n_pix - 9
            w[:, 0] = 0x0800 | (no % 100)
            w[:, 1] = 0xC000 | (no & 0x3FFF)
            w[:, 2], w[:, 3] = total >> 16, total & 0xFFFF
            w[:, 4], w[:, 5] = 0x10D2, 0x0100 | t
            w[:, 6], w[:, 7] = 0x6553, no >> 4
            w[:, 8] = (no * 641) & 0xFFFF
            w[:, 9], w[:, 10], w[:, 11] = cam.n_pix, cam.n_samp, cam.n_gain << 8
            w[:, 14], w[:, 15] = no >> 16, no & 0xFFFF
            body = view[a:a + n, :, :, :cam.n_pix].reshape(n, -1).to(torch.int32) & 0xFFFF
            words = torch.cat([w, body], 1)
            words = torch.cat([words, _crc16(words)[:, None]], 1)
            words = ((words & 0xFF) << 8 | words >> 8).to(torch.int16)  # big-endian in the stream
            at = torch.from_numpy(off[part] // 2).to(DEV)[:, None] + torch.arange(words.shape[1], device=DEV)
            buf[at.reshape(-1)] = words.reshape(-1)
    return cams, types, buf.view(torch.uint8), off, slot


# ---------------------------------------------------------------------------
# What a program holds before the call, and the call
# ---------------------------------------------------------------------------
def _record_parts(rec):
    """The columns of image-parameter records, by kind."""
    size, cog, axes, psi, moments, times, edge, counts = rec.split((1, 2, 2, 1, 2, 2, 2, 4), dim=1)
    return {"size": size, "cog": cog, "axes": axes, "psi": psi, "moments": moments, "times": times, "edge": edge,
            "counts": counts.view(torch.int32)}


def prepare(case, seed):
    op = case["op"]
    if op == "reconstruct":
        cams, types, ev_off, pool, off, _ = _traces(case, seed)
        handles = [c.handle() for c in cams]
        pipe = rta.Pipeline(handles, do_stereo=ev_off is not None, extractor=EXTRACTORS[case["extractor"]])
        mlp = None
        if case["classify"] != "none":
            mlp = _mlp(seed)
            pipe.attach_mlp(mlp, _boxcut())
        cls = torch.empty((len(types), 2), dtype=torch.float32, device=DEV) if case["classify"] == "camera" else None
        batch = pipe.make_batch(pool.view(torch.uint16), torch.from_numpy(types).to(DEV),
                                torch.from_numpy(off).to(DEV),
                                None if ev_off is None else torch.from_numpy(ev_off).to(DEV), tel_class=cls)
        tel, evt = pipe.alloc_outputs(batch, torch.device(DEV))
        out = {"images": _record_parts(tel)}
        if cls is not None:
            out["class"] = cls
        if evt is not None:
            d, cond, ge, counts = evt.split((2, 1, 2, 3), dim=1)
            out["events"] = {"dir": d, "cond": cond, "class": ge, "counts": counts.view(torch.int32)}
        return {"op": op, "pipe": pipe, "mlp": mlp, "batch": batch, "tel": tel, "evt": evt, "out": out}
    if op == "stages":
        cams, _, _, pool, _, _ = _traces(case, seed)
        return {"op": op, "cam": cams[0].handle(), "traces": pool.view(torch.uint16)}
    if op == "health":
        cams, _, _, pool, _, _ = _traces(case, seed, signal=False)
        return {"op": op, "cam": cams[0].handle(), "traces": pool.view(torch.uint16)}
    if op == "packets":
        cams, types, data, off, slot = _stream(case, seed)
        pipe = rta.Pipeline([c.handle() for c in cams], do_stereo=False)
        pool = torch.zeros(max(int(slot[-1]), 8), dtype=torch.uint16, device=DEV)
        return {"op": op, "pipe": pipe, "data": data, "n_bytes": int(off[-1]),
                "pkt_off": torch.from_numpy(off[:-1].copy()).to(DEV), "tel_type": torch.from_numpy(types).to(DEV),
                "slot": torch.from_numpy(slot[:-1].copy()).to(DEV), "elems": int(slot[-1]), "pool": pool,
                "view": pool.view(torch.int16)}
    if op == "alerts":
        evt, t = _sky(case, seed)
        sam = rta.Sam(case["grid"], 3600, 0.0, 1.0, 0.0015, 1.5, 3.5, 7.0, 0.7, 5.0, list(SCALES))
        return {"op": op, "sam": sam, "evt": evt, "t": t}
    if op == "train":
        x, label, log10e, rows = _training_set(case, seed)
        loss = torch.zeros(case["steps"], dtype=torch.float32, device=DEV)
        return {"op": op, "mlp": _mlp(seed, case["batch"]), "x": x, "label": label, "log10e": log10e, "rows": rows,
                "loss": loss, "slots": [loss[i:i + 1] for i in range(case["steps"])]}
    if op == "classify":
        return {"op": op, "mlp": _mlp(seed), "bc": _boxcut(), "rec": _image_records(case["records"], seed)}
    raise ValueError("unknown op %r" % op)


def run(state):
    s, op = state, state["op"]
    if op == "reconstruct":
        s["pipe"].process(s["batch"], s["tel"], s["evt"])
        return s["out"]
    if op == "stages":
        out = rta.calibrate(s["cam"], s["traces"])
        mask = rta.clean(s["cam"], out["D"], out["gain"])
        rec = rta.hillas(s["cam"], out["q"], out["t"], mask, out["gain"])
        return {"pixels": out, "mask": mask, "images": _record_parts(rec)}
    if op == "packets":
        pool, rec = rta.decode_packets(s["pipe"], s["data"], s["pkt_off"], s["tel_type"], s["slot"], s["elems"],
                                       pool=s["pool"], n_bytes=s["n_bytes"])
        return {"pool": s["view"], "records": rec.view(torch.int32), "types": s["tel_type"]}
    if op == "health":
        pix, cam = rta.health(s["cam"], s["traces"], to_host=False)
        sums, moments, flags = pix.split((4, 2, 2), dim=1)
        return {"sums": sums.view(torch.int64), "moments": moments, "flags": flags.view(torch.int64),
                "median": cam[:s["cam"].n_gain], "verdict": cam[2:].view(torch.int64)}
    if op == "alerts":
        s["sam"].clear()
        s["sam"].fill(s["evt"], s["t"])
        sig, n_on, n_off, _, found = s["sam"].search(3599)
        return {"significance": sig, "n_on": n_on, "n_off": n_off, "alerts": found}
    if op == "train":
        for rows, slot in zip(s["rows"], s["slots"]):
            s["mlp"].train_step(s["x"], s["label"], s["log10e"], loss_out=slot, rows=rows)
        return {"loss": s["loss"], "params": s["mlp"].get_params()}
    return rta.classify(s["mlp"], s["bc"], s["rec"])


def work(case):
    op = case["op"]
    row_flops = 2.0 * (10 * 64 + 2 * 64 * 64 + 64 * 2)
    if op in ("reconstruct", "stages", "packets", "health"):
        cams, _ = _cameras(case["cameras"])
        types, ev_off = _layout(case)
        count = np.bincount(types, minlength=len(cams))
        one_gain = sum(int(n) * c.n_pix * c.n_samp * 2 for n, c in zip(count, cams))
        pixels = sum(int(n) * c.n_pix for n, c in zip(count, cams))
        both = sum(int(n) * c.n_pix * c.n_samp * c.n_gain * 2 for n, c in zip(count, cams))
        n = len(types)
    if op == "reconstruct":
        # the high gain once (four samples of it for the fixed window), records and descriptors
        b = (8 * pixels if case["extractor"] == "fixed" else one_gain) + n * 76
        f = 3.0 * (4 * pixels if case["extractor"] == "fixed" else one_gain / 2)
        if case["classify"] != "none":
            b += 8 * n if case["classify"] == "camera" else 0
            f += n * row_flops
        if ev_off is not None:
            b += 40 * (len(ev_off) - 1)
        return {"bytes": b, "flops": f}
    if op == "stages":
        # traces in; 19 bytes per pixel of calibrated products, the mask and the records out
        return {"bytes": one_gain + 20 * pixels + 64 * n, "flops": 1.5 * one_gain}
    if op == "packets":
        pool = sum(int(k) * c.elems * 2 for k, c in zip(count, cams))
        return {"bytes": both + pool + n * (34 + 32 + 20), "flops": both / 2}
    if op == "health":
        return {"bytes": both + 64 * sum(c.n_pix * c.n_gain for c in cams), "flops": 2.0 * both}
    if op == "alerts":
        cube, maps = 3600 * case["grid"] ** 2 * 4, len(SCALES) * case["grid"] ** 2 * 16
        return {"bytes": 40 * case["events"] + 2 * cube + maps, "flops": 10.0 * case["events"]}
    if op == "train":
        return {"bytes": case["steps"] * (case["batch"] * 56 + 9154 * 4 * 7),
                "flops": case["steps"] * case["batch"] * 3.0 * row_flops}
    return {"bytes": 80 * case["records"], "flops": case["records"] * row_flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch and numpy
# ---------------------------------------------------------------------------
def _pixels_exact(cam, tr, extractor):
    """Calibration of traces int16 [n][G][T][Npad]: dict of int64 / float64 [n][N]."""
    n, T, N = tr.shape[0], cam.n_samp, cam.n_pix
    x = tr[:, :, :, :N].to(torch.int32) & 0xFFFF
    c = torch.cumsum(x, 2, dtype=torch.int32)
    W = c[:, :, WINDOW - 1:].clone()
    W[:, :, 1:] -= c[:, :, :-WINDOW]
    n_start = W.shape[2]
    rank = (255 - torch.arange(n_start, device=DEV, dtype=torch.int32))
    low = torch.zeros((n, N), dtype=torch.bool, device=DEV)
    s0 = (T - WINDOW) // 2
    if cam.n_gain == 2:
        seen = x[:, 0, s0:s0 + WINDOW] if extractor == "fixed" else x[:, 0]
        low = seen.amax(1) >= SWITCH_ADC
    if extractor == "fixed":
        s = torch.full((n, N), s0, dtype=torch.int64, device=DEV)
    elif extractor == "global":
        key = W[:, 0].sum(2, dtype=torch.int64) * 256 + rank[None, :]
        s = (255 - key.amax(1) % 256)[:, None].expand(n, N)
    elif extractor == "neighbour":
        padded = torch.cat([W[:, 0], torch.zeros_like(W[:, 0, :, :1])], 2)
        nbr = torch.from_numpy(np.where(cam.nbr < 0, N, cam.nbr).astype(np.int64)).to(DEV)
        total = sum(padded[:, :, nbr[:, k]] for k in range(6))
        s = 255 - (total * 256 + rank[None, :, None]).amax(1).long() % 256
    else:
        best = (W * 256 + rank[None, None, :, None]).amax(2)
        s = 255 - (torch.where(low, best[:, -1], best[:, 0]).long() % 256)
    g = low.long() * (cam.n_gain - 1)
    ev, pix = torch.arange(n, device=DEV)[:, None], torch.arange(N, device=DEV)[None]
    samples = torch.stack([x[ev, g, s + k, pix] for k in range(WINDOW)], 0).long()
    P = torch.from_numpy(np.rint(256.0 * cam.ped.astype(np.float64)).astype(np.int64)).to(DEV)[g, pix]
    adc = torch.from_numpy(cam.adc.astype(np.float64)).to(DEV)
    S = samples.sum(0)
    D = 256 * S - WINDOW * P
    nt = sum(k * (256 * samples[k] - P) for k in range(WINDOW))
    t = s + torch.where(D > 0, nt.double() / D.clamp(min=1).double(), torch.full_like(nt.double(), 1.5))
    first = (samples * 8 + torch.arange(7, 7 - WINDOW, -1, device=DEV)[:, None, None]).amax(0)
    pic, bnd = (torch.ceil(256.0 * adc * v)[g, pix] for v in (T_PIC, T_BND))
    return {"S": S, "D": D, "sstar": s, "peak": s + 7 - first % 8, "gain": low.long(), "q": D.double() / (256.0 * adc[g, pix]),
            "t": t, "pic": D >= pic, "bnd": D >= bnd}


def _mask_exact(cam, p):
    N = cam.n_pix
    nbr = torch.from_numpy(np.where(cam.nbr < 0, N, cam.nbr).astype(np.int64)).to(DEV)

    def near(v):
        v = torch.cat([v, torch.zeros_like(v[:, :1])], 1)
        return functools.reduce(torch.logical_or, (v[:, nbr[:, k]] for k in range(6)))

    return (p["bnd"] & near(p["pic"])) | (p["pic"] & near(p["bnd"]))


def _image_exact(cam, p, mask):
    """Image parameters [n][12] float64 and counts [n][4] of masked pixels."""
    n, N = mask.shape
    x, y = (torch.from_numpy(v.astype(np.float64)).to(DEV)[None] for v in (cam.x, cam.y))
    q = torch.where(mask, p["q"], 0.0)
    m = mask.double()
    cnt, S = mask.sum(1), q.sum(1)
    xm, ym = (q * x).sum(1) / S, (q * y).sum(1) / S
    dx, dy = x - xm[:, None], y - ym[:, None]
    sxx, syy, sxy = ((q * a * b).sum(1) / S for a, b in ((dx, dx), (dy, dy), (dx, dy)))
    hd = 0.5 * (sxx - syy)
    length = torch.sqrt(0.5 * (sxx + syy) + torch.sqrt(hd * hd + sxy * sxy))
    psi = 0.5 * torch.atan2(2 * sxy, sxx - syy)
    psi = torch.where(psi <= -math.pi / 2, psi + math.pi, psi)
    lon = dx * torch.cos(psi)[:, None] + dy * torch.sin(psi)[:, None]
    tra = dy * torch.cos(psi)[:, None] - dx * torch.sin(psi)[:, None]
    width = torch.sqrt((q * tra * tra).sum(1) / S)
    skew, kurt = ((q * lon ** k).sum(1) / (S * length ** k) for k in (3, 4))
    lbar, tbar = (m * lon).sum(1) / cnt, (m * p["t"]).sum(1) / cnt
    dl = lon - lbar[:, None]
    grad = (m * dl * (p["t"] - tbar[:, None])).sum(1) / (m * dl * dl).sum(1)
    border = torch.from_numpy((cam.nbr >= 0).sum(1) < 6).to(DEV)
    leak = (q * border).sum(1) / S
    rec = torch.stack([S, xm, ym, length, width, psi, skew, kurt, grad, tbar - grad * lbar, leak,
                       torch.sqrt(xm * xm + ym * ym)], 1)
    good = (cnt >= 2) & (S > 0)
    rec[:, 1:] = torch.where(good[:, None], rec[:, 1:], math.nan)
    # islands: the smallest pixel index spreads over each connected component
    nbr = torch.from_numpy(np.where(cam.nbr < 0, N, cam.nbr).astype(np.int64)).to(DEV)
    own = torch.arange(N, device=DEV)[None].expand(n, N)
    lab = torch.where(mask, own, N)
    while True:
        pad = torch.cat([lab, torch.full_like(lab[:, :1], N)], 1)
        new = functools.reduce(torch.minimum, (pad[:, nbr[:, k]] for k in range(6)), lab)
        new = torch.where(mask, new, N)
        if torch.equal(new, lab):
            break
        lab = new
    n_low = p["gain"].sum(1)
    flags = (n_low > 0).long() * rta.FLAG_LOW_GAIN + (~good).long() * (rta.FLAG_HILLAS_INVALID | rta.FLAG_TIME_INVALID)
    return rec, torch.stack([cnt, (mask & (lab == own)).sum(1), n_low, flags], 1)


def _images_exact(cam, tr, extractor="sliding"):
    recs, counts = [], []
    step = max(1, int(24e6 / (cam.n_gain * cam.n_samp * cam.n_pad)))
    for a in range(0, len(tr), step):
        p = _pixels_exact(cam, tr[a:a + step], extractor)
        r, c = _image_exact(cam, p, _mask_exact(cam, p))
        recs.append(r)
        counts.append(c)
    return torch.cat(recs), torch.cat(counts)


def _parts64(rec, counts):
    size, cog, axes, psi, moments, times, edge = rec.split((1, 2, 2, 1, 2, 2, 2), dim=1)
    return {"size": size, "cog": cog, "axes": axes, "psi": psi, "moments": moments, "times": times, "edge": edge,
            "counts": counts}


def _features64(rec, counts):
    return torch.stack([torch.log10(rec[:, 0]), rec[:, 3], rec[:, 4], rec[:, 11], rec[:, 5], rec[:, 6], rec[:, 7],
                        rec[:, 8], rec[:, 10], counts[:, 1].double()], 1)


def _layers64(params):
    w = torch.as_tensor(np.asarray(params, np.float64), device=DEV)
    out, at = [], 0
    for n_in, n_out in ((10, 64), (64, 64), (64, 64), (64, 2)):
        out.append((w[at:at + n_in * n_out].view(n_in, n_out), w[at + n_in * n_out:at + (n_in + 1) * n_out]))
        at += (n_in + 1) * n_out
    return out


def _forward64(layers, feat):
    h = (feat - torch.from_numpy(FEAT_MEAN).to(DEV).double()) / torch.from_numpy(FEAT_STD).to(DEV).double()
    for k, (w, b) in enumerate(layers):
        h = h @ w + b
        if k < 3:
            h = torch.relu(h)
    return h


def _decide64(seed, feat):
    """[score, log10 E, gamma, fallback] of feature rows."""
    bc = _boxcut()
    lo, hi = torch.from_numpy(FEAT_LO).to(DEV).double(), torch.from_numpy(FEAT_HI).to(DEV).double()
    inside = (torch.isfinite(feat) & (feat >= lo) & (feat <= hi)).all(1)
    o = _forward64(_layers64(_network(seed)), torch.nan_to_num(feat, 0.0, 0.0, 0.0))
    score = torch.sigmoid(o[:, 0])
    b = torch.floor(torch.nan_to_num(feat[:, 0] - bc.lgs_lo) / (bc.lgs_hi - bc.lgs_lo) * bc.n_bins).long()
    b = b.clamp(0, bc.n_bins - 1)
    tab = {k: torch.tensor(list(getattr(bc, k)), device=DEV).double()[b] for k in ("w_mean", "w_std", "l_mean", "l_std")}
    box = ((feat[:, 2] - tab["w_mean"]) / tab["w_std"] < bc.cut_w) & ((feat[:, 1] - tab["l_mean"]) / tab["l_std"] < bc.cut_l)
    return torch.stack([torch.where(inside, score, box.double()),
                        torch.where(inside, o[:, 1], bc.e_a + bc.e_b * feat[:, 0]),
                        torch.where(inside, score > bc.mlp_cut, box).double(), (~inside).double()], 1)


def _reconstruct_exact(case, seed):
    cams, types, ev_off, _, _, groups = _traces(case, seed)
    n = len(types)
    rec = torch.zeros((n, 12), dtype=torch.float64, device=DEV)
    counts = torch.zeros((n, 4), dtype=torch.int64, device=DEV)
    for cam, (idx, tr) in zip(cams, groups):
        if len(idx):
            i = torch.from_numpy(idx).to(DEV)
            rec[i], counts[i] = _images_exact(cam, tr, case["extractor"])
    valid = (counts[:, 3] & rta.FLAG_HILLAS_INVALID) == 0
    cls = None
    if case["classify"] != "none":
        d = _decide64(seed, _features64(rec, counts))
        counts[:, 3] |= (valid & (d[:, 3] > 0)).long() * rta.FLAG_MLP_FALLBACK
        cls = torch.where(valid[:, None], d[:, :2], math.nan)
    out = {"images": _parts64(rec, counts)}
    if case["classify"] == "camera":
        out["class"] = cls
    if ev_off is not None:
        focal = torch.tensor([c.focal for c in cams], dtype=torch.float64, device=DEV)[torch.from_numpy(types).to(DEV).long()]
        mult = torch.from_numpy(np.diff(ev_off)).to(DEV)
        e = torch.repeat_interleave(torch.arange(len(mult), device=DEV), mult)
        ratio = rec[:, 4] / rec[:, 3]
        use = valid & (rec[:, 3] > 0) & (ratio <= 0.9)
        w = torch.where(use, rec[:, 0] * (1 - ratio), 0.0)
        nx, ny = -torch.sin(rec[:, 5]), torch.cos(rec[:, 5])
        nc = nx * rec[:, 1] / focal + ny * rec[:, 2] / focal

        def total(v, on):
            return torch.zeros(len(mult), dtype=torch.float64, device=DEV).index_add_(0, e, torch.where(on, v, 0.0))

        A00, A01, A11, b0, b1 = (total(w * v, use) for v in (nx * nx, nx * ny, ny * ny, nc * nx, nc * ny))
        used = total(torch.ones_like(w), use)
        det = A00 * A11 - A01 * A01
        lmax = 0.5 * (A00 + A11) + torch.sqrt(0.25 * (A00 - A11) ** 2 + A01 * A01)
        good = (used >= 2) & (lmax < 1e4 * (det / lmax))
        d = torch.where(good[:, None], torch.stack([(A11 * b0 - A01 * b1) / det, (A00 * b1 - A01 * b0) / det], 1), math.nan)
        ge = torch.full((len(mult), 2), math.nan, dtype=torch.float64, device=DEV)
        if cls is not None:
            size = torch.where(valid, rec[:, 0], 0.0)
            s = total(size, valid)
            ge = torch.stack([total(size * cls[:, k], valid) / s for k in (0, 1)], 1)
        # the condition number of near-parallel axes holds no digits in 32 bits
        out["events"] = {"dir": d, "cond": None, "class": ge, "counts": None}
    return out


def _alerts_exact(case, seed):
    evt, t = (v.cpu().numpy() for v in _sky(case, seed))
    G, cell = case["grid"], float(np.float32(0.0015))
    ok = (evt.view(np.int32)[:, 7] & rta.EVT_STEREO_INVALID == 0) & (evt[:, 3] >= np.float32(0.7))
    b = np.floor(t[ok]).astype(np.int64)
    ix, iy = (np.floor(evt[ok, k].astype(np.float64) / cell + 0.5 * G).astype(np.int64) for k in (0, 1))
    inside = (b >= 0) & (b < 3600) & (ix >= 0) & (ix < G) & (iy >= 0) & (iy < G)
    cube = np.bincount((b[inside] * G + iy[inside]) * G + ix[inside], minlength=3600 * G * G).reshape(3600, G, G)
    d2 = np.add.outer(np.arange(-7, 8) ** 2, np.arange(-7, 8) ** 2)
    sig, on_maps, off_maps = [], [], []

    def spread(m, ker):
        out, pad = np.zeros((G, G), np.int64), np.pad(m, 7)
        for j, i in zip(*np.nonzero(ker)):
            out += pad[j:j + G, i:i + G]
        return out

    near, ring = d2 <= 1.5 ** 2, (d2 > 3.5 ** 2) & (d2 <= 7.0 ** 2)
    c_on, c_off = spread(np.ones((G, G), np.int64), near), spread(np.ones((G, G), np.int64), ring)
    for w in SCALES:
        m = cube[3600 - w:].sum(0)
        on, off = spread(m, near), spread(m, ring)
        a = c_on / c_off
        with np.errstate(divide="ignore", invalid="ignore"):
            t1 = np.where(on > 0, on * np.log((1 + a) / a * on / (on + off)), 0.0)
            t2 = np.where(off > 0, off * np.log((1 + a) * off / (on + off)), 0.0)
        s = np.copysign(np.sqrt(np.maximum(2 * (t1 + t2), 0.0)), on - a * off)
        sig.append(np.where(on * c_off == c_on * off, 0.0, s))
        on_maps.append(on)
        off_maps.append(off)
    sig = np.stack(sig)
    return {"significance": sig, "n_on": np.stack(on_maps), "n_off": np.stack(off_maps), "alerts": int((sig >= 5.0).sum())}


def _train_exact(case, seed):
    x, label, log10e, rows = _training_set(case, seed)
    p = torch.as_tensor(_network(seed).astype(np.float64), device=DEV).requires_grad_(True)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    losses = []
    for k, r in enumerate(rows):
        layers, at = [], 0
        for n_in, n_out in ((10, 64), (64, 64), (64, 64), (64, 2)):
            layers.append((p[at:at + n_in * n_out].view(n_in, n_out), p[at + n_in * n_out:at + (n_in + 1) * n_out]))
            at += (n_in + 1) * n_out
        o = _forward64(layers, x[r].double())
        lab, y = label[r].double(), log10e[r].double()
        z = o[:, 0]
        loss = (torch.relu(z) - z * lab + torch.log1p(torch.exp(-z.abs())) + lab * (o[:, 1] - y) ** 2).mean()
        g, = torch.autograd.grad(loss, p)
        losses.append(loss.detach())
        with torch.no_grad():
            m = b1 * m + (1 - b1) * g
            v = b2 * v + (1 - b2) * g * g
            p -= float(np.float32(1e-3)) * (m / (1 - b1 ** (k + 1))) / (torch.sqrt(v / (1 - b2 ** (k + 1))) + 1e-8)
    return {"loss": torch.stack(losses), "params": p.detach()}


def exact(case, seed):
    op = case["op"]
    if op == "reconstruct":
        return _reconstruct_exact(case, seed)
    if op == "stages":
        cams, _, _, _, _, groups = _traces(case, seed)
        cam, tr = cams[0], groups[0][1]
        pix, masks, recs, counts = {}, [], [], []
        step = max(1, int(24e6 / (cam.n_gain * cam.n_samp * cam.n_pad)))
        for a in range(0, len(tr), step):
            p = _pixels_exact(cam, tr[a:a + step], "sliding")
            mask = _mask_exact(cam, p)
            r, c = _image_exact(cam, p, mask)
            masks.append(mask.long())
            recs.append(r)
            counts.append(c)
            for k in ("S", "D", "sstar", "peak", "gain", "q", "t"):
                pix.setdefault(k, []).append(p[k])
        return {"pixels": {k: torch.cat(v) for k, v in pix.items()}, "mask": torch.cat(masks),
                "images": _parts64(torch.cat(recs), torch.cat(counts))}
    if op == "health":
        cams, _, _, _, _, groups = _traces(case, seed, signal=False)
        cam, tr = cams[0], groups[0][1]
        mean, rms = [], []
        for g in range(cam.n_gain):
            s1 = torch.zeros(cam.n_pix, dtype=torch.int64, device=DEV)
            s2 = torch.zeros_like(s1)
            for a in range(0, len(tr), 64):
                v = tr[a:a + 64, g, :, :cam.n_pix].to(torch.int64) & 0xFFFF
                s1 += v.sum((0, 1))
                s2 += (v * v).sum((0, 1))
            n = float(len(tr) * cam.n_samp)
            mean.append(s1.double() / n)
            rms.append(torch.sqrt((s2.double() / n - mean[-1] ** 2).clamp(min=0)))
        median = torch.stack([torch.sort(r).values[(cam.n_pix - 1) // 2] for r in rms])
        return {"sums": None, "moments": torch.stack([torch.cat(mean), torch.cat(rms)], 1), "flags": None,
                "median": median, "verdict": None}
    if op == "alerts":
        return _alerts_exact(case, seed)
    if op == "train":
        return _train_exact(case, seed)
    if op == "classify":
        rec = _image_records(case["records"], seed)
        return _decide64(seed, _features64(rec[:, :12].double(), rec.view(torch.int32)[:, 12:].long()))
    return None  # packets: whole numbers
