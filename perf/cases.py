"""The calls that a dedispersion program makes of this package, as timed cases.

A case is one pass of one kind of work:

  tree       a z-scored filterbank block is encoded (or cast) to the plan's storage type and
             dedispersed; with "detect" the plane also goes through the matched filter and the
             candidate stage.
  detect     the matched filter and candidate stage alone, on a float plane.
  stream     one arrival of a chunk for every beam of a server: encode or cast, batched push
             through the history rings, batched detection.
  frontend   raw power to encoder bits: clipped statistics, normalisation, channel flagging,
             zero-DM subtraction, encoder.
  multirate  a whole search of a block: scrunch bands, re-encoded trees, detection, merge.
  fdmt       the FDMT transform of a block.

Sizes are those of the repository's workloads (a 64-channel beam of 64 or 3000 trial DMs, the
1024-channel beam of 4096 trial DMs, 8192-sample chunks) and sizes between them, odd ones included.
The instrument is the workloads': 16 MHz below 416 MHz, 0.138 ms sampling.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2606_15361_amd as snd
from paper_2606_15361_amd.serve import Server

KDM_MS = 4.148808e6        # dispersion constant, MHz^2 ms per (pc cm^-3)
TSAMP_S = 0.138e-3
F_HI, BAND = 416.0, 16.0   # MHz
SWEEP_PER_DM = 14.17       # samples the whole band sweeps per unit of DM
WIDTHS = (1, 2, 4, 8, 16, 32, 64)
WIDTHS_SCALED = tuple(1 << i for i in range(11))   # 1 .. 1024, the DM-scaled set
THRESHOLDS = (1.0, 2.0, 3.0, 4.0)                  # graded encoder, in sigma
TABLE = 512                # candidates kept per pass, in (DM, time) order


# ------------------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest beam of the workloads, binary on bit rows, encoded, dedispersed and searched:
        # a few launches and one read-back, so latency and host work decide
        dict(name="tree_bits_64ch", kind="tree", mode="bits", nchan=64, nsamp=8192, ndm=64, dm_max=300.0, grid="linear",
             branching=2, detect=True, time_major=False),
        # the 64-channel beam over a geometric grid of 3000 DMs to 2000, graded, with its search:
        # neighbouring DMs lie far apart, so they share little
        dict(name="tree_graded_64ch", kind="tree", mode="graded", nchan=64, nsamp=65536, ndm=3000, dm_max=2000.0,
             grid="geometric", branching=4, detect=True, time_major=False),
        # the same grid in float
        dict(name="tree_f32_64ch", kind="tree", mode="f32", nchan=64, nsamp=65536, ndm=3000, dm_max=2000.0,
             grid="geometric", branching=4, detect=False, time_major=False),
        # the headline block: 1024 channels, 4096 DMs, 2^17 samples, float32
        dict(name="tree_f32_1024ch", kind="tree", mode="f32", nchan=1024, nsamp=1 << 17, ndm=4096, dm_max=2000.0,
             grid="linear", branching=4, detect=False, time_major=False),
        # the same block graded, from the time-major order that recorders write, with its search
        dict(name="tree_graded_1024ch", kind="tree", mode="graded", nchan=1024, nsamp=1 << 17, ndm=4096, dm_max=2000.0,
             grid="linear", branching=4, detect=True, time_major=True),
        # the same block binary on bit rows, with its search
        dict(name="tree_bits_1024ch", kind="tree", mode="bits", nchan=1024, nsamp=1 << 17, ndm=4096, dm_max=2000.0,
             grid="linear", branching=4, detect=True, time_major=False),
        # a channel count that leaves every level of the tree ragged, an odd DM count and length
        dict(name="tree_graded_1000ch", kind="tree", mode="graded", nchan=1000, nsamp=40013, ndm=1021, dm_max=500.0,
             grid="linear", branching=4, detect=False, time_major=False),
        # the search of a large float plane with the DM-scaled width set (1 .. 1024 samples)
        dict(name="detect_f32", kind="detect", ndm=4096, n_out=102748, scaled=True, sigma="std"),
        # serving: eight beams, half graded and half float stored in bf16, one 8192-sample chunk each
        dict(name="stream_8beams", kind="stream", nchan=1024, chunk=8192, ndm=4096, dm_max=2000.0, beams=8),
        # raw power of the large beam to encoder bits
        dict(name="frontend_1024ch", kind="frontend", nchan=1024, nsamp=1 << 17, window=8192),
        # a whole multi-rate search of the large block, graded
        dict(name="multirate_graded", kind="multirate", nchan=1024, nsamp=1 << 17, ndm=4096, dm_max=2000.0),
        # the FDMT of a block half as long, to half the DM
        dict(name="fdmt_1024ch", kind="fdmt", nchan=1024, nsamp=1 << 16, dm_max=1000.0),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, even in its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dm_for(rng, nsamp, top=2000.0):
    """A largest DM whose sweep takes 15 to 65 per cent of a block."""
    return round(min(top, rng.uniform(0.15, 0.65) * nsamp / SWEEP_PER_DM), 1)


def draw(rng):
    kind = rng.choice(["tree"] * 7 + ["detect", "stream", "frontend", "multirate", "fdmt"])
    if kind == "tree":
        mode = rng.choice(["f32", "bf16", "f16", "graded", "bits"])
        ragged = rng.random() < 0.4
        nchan = _log(rng, 64, 1024) if ragged else 1 << rng.randint(6, 10)
        nsamp = _log(rng, 6000, 1 << 17)
        # trees of irregular nodes in the integer modes stay small, as the workloads keep them
        ndm = _log(rng, 40, 1000 if ragged and mode in ("graded", "bits") else 4096)
        branching = rng.choice([2, 4, 4, 8])
        return dict(kind="tree", mode=mode, nchan=nchan, nsamp=nsamp, ndm=ndm, dm_max=_dm_for(rng, nsamp),
                    grid=rng.choice(["linear", "linear", "geometric"]) if nchan <= 128 else "linear",
                    branching=branching, detect=mode in ("graded", "bits") and rng.random() < 0.5,
                    time_major=mode in ("graded", "bits") and rng.random() < 0.3)
    if kind == "detect":
        return dict(kind="detect", ndm=_log(rng, 64, 4096), n_out=_log(rng, 3000, 100000), scaled=rng.random() < 0.5,
                    sigma="mad" if rng.random() < 0.25 else "std")
    if kind == "stream":
        return dict(kind="stream", nchan=1 << rng.randint(6, 10), chunk=_log(rng, 2000, 8192), ndm=_log(rng, 200, 4096),
                    dm_max=round(rng.uniform(100.0, 2000.0), 1), beams=rng.randint(1, 8))
    if kind == "frontend":
        return dict(kind="frontend", nchan=_log(rng, 64, 1024), nsamp=_log(rng, 8192, 1 << 17),
                    window=rng.choice([2048, 4096, 8192]))
    if kind == "multirate":
        return dict(kind="multirate", nchan=1 << rng.randint(6, 10), nsamp=_log(rng, 50000, 1 << 17),
                    ndm=_log(rng, 500, 4096), dm_max=round(rng.uniform(800.0, 2000.0), 1))
    nsamp = _log(rng, 6000, 1 << 16)
    return dict(kind="fdmt", nchan=1 << rng.randint(6, 10), nsamp=nsamp, dm_max=_dm_for(rng, nsamp, 1000.0))


# ------------------------------------------------------------------------------- inputs

def _freqs(nchan):
    return F_HI - (np.arange(nchan, dtype=np.float64) + 0.5) * BAND / nchan


def _dms(case):
    n, top = case["ndm"], case["dm_max"]
    if case.get("grid", "linear") == "linear":
        return np.linspace(0.0, top, n, dtype=np.float64)
    knee = 100.0  # the step grows in proportion to DM + knee
    return knee * (((top + knee) / knee) ** (np.arange(n) / max(1, n - 1)) - 1.0)


def _delays(freqs, dms, tsamp_s=TSAMP_S):
    """Whole-sample delays [ndm][nchan] against the highest channel."""
    inv = 1.0 / (freqs * freqs) - 1.0 / (freqs.max() ** 2)
    return np.rint((KDM_MS * dms)[:, None] * inv[None, :] / (tsamp_s * 1e3)).astype(np.int64)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _filterbank(seed, nchan, nsamp, dm_max, npulses=6):
    """Gaussian noise with dispersed pulses of 1 to 40 samples, float32 [nchan][nsamp]."""
    z = torch.randn((nchan, nsamp), generator=_gen(seed), device="cuda", dtype=torch.float32)
    rng = np.random.default_rng(seed)
    f = _freqs(nchan)
    for _ in range(npulses):
        w = int(np.exp(rng.uniform(0.0, math.log(40.0))))
        d = _delays(f, np.array([dm_max * rng.uniform(0.1, 0.95)]))[0]
        t0 = int(rng.uniform(0.0, max(1.0, nsamp - d.max() - w)))
        at = np.minimum(t0 + d[:, None] + np.arange(w)[None, :], nsamp - 1)
        amp = float(rng.uniform(12.0, 40.0) / math.sqrt(w * nchan))
        rows = torch.arange(nchan, device="cuda")[:, None].expand(nchan, w)
        z.index_put_((rows, torch.from_numpy(at).cuda()), torch.tensor(amp, device="cuda"), accumulate=True)
    return z


def _plan(case):
    mode = case["mode"]
    kw = dict(branching=case["branching"])
    if mode in ("f32", "bf16", "f16"):
        kw.update(mode="float", in_dtype=mode, node_dtype=mode)
    elif mode == "graded":
        kw.update(mode="graded")
    else:
        kw.update(mode="binary", k_leaf=2, k_int=1)
        kw.update(in_dtype="bits")
    try:
        p = snd.Plan(_freqs(case["nchan"]), _dms(case), TSAMP_S, case["nsamp"], **kw)
    except snd.SndError:  # bit input needs bit rows, whose level-1 nodes are all of one fan-in
        kw.pop("in_dtype", None)
        p = snd.Plan(_freqs(case["nchan"]), _dms(case), TSAMP_S, case["nsamp"], **kw)
    p.upload("cuda")
    return p


def _power(case, seed):
    """Raw power: exponential noise, one gain per channel, some loud channels, broadband bursts."""
    nchan, nsamp = case["nchan"], case["nsamp"]
    g = _gen(seed)
    p = torch.empty((nchan, nsamp), device="cuda").exponential_(generator=g)
    p *= 0.5 + torch.rand((nchan, 1), generator=g, device="cuda")
    rng = np.random.default_rng(seed)
    for c in rng.choice(nchan, size=max(1, nchan // 64), replace=False):  # interference for part of the block
        a = int(rng.integers(0, nsamp // 2))
        p[int(c), a:a + nsamp // 4] *= 4.0
    for t in rng.choice(nsamp, size=8, replace=False):
        p[:, int(t)] += 2.0
    return p


def prepare(case, seed):
    kind = case["kind"]
    if kind == "tree":
        p = _plan(case)
        z = _filterbank(seed, case["nchan"], case["nsamp"], case["dm_max"])
        s = dict(case=case, plan=p, z=z.t().contiguous() if case["time_major"] else z, out=p.empty_output("cuda"))
        p.workspace("cuda")
        if case["detect"]:
            s["det"] = snd.Detector(p, widths=WIDTHS, max_pixels=1 << 22)
        return s
    if kind == "detect":
        # any plan of this shape carries the plane's sizes; its DM grid gives the width sets
        dm = min(2000.0, 0.4 * case["n_out"] / SWEEP_PER_DM)
        f, dms = _freqs(16), np.linspace(0.0, dm, case["ndm"])
        p = snd.Plan(f, dms, TSAMP_S, case["n_out"] + int(_delays(f, dms).max()), mode="float")
        y = p.empty_output("cuda")
        y.normal_(0.0, 32.0, generator=_gen(seed))
        rng = np.random.default_rng(seed)
        for _ in range(12):  # pulses, brightest at their DM and fading over its neighbours
            k, t, w = int(rng.integers(0, p.ndm)), int(rng.integers(0, max(1, p.n_out - 200))), int(rng.integers(1, 100))
            for dk in range(-6, 7):
                if 0 <= k + dk < p.ndm:
                    y[k + dk, t:t + w] += float(rng.uniform(8.0, 14.0)) * 32.0 / math.sqrt(w) / (1.0 + 0.3 * abs(dk))
        kw = dict(n_base_widths=4, width_alpha=0.1) if case["scaled"] else {}
        det = snd.Detector(p, widths=WIDTHS_SCALED if case["scaled"] else WIDTHS, sigma=case["sigma"], **kw)
        return dict(case=case, plan=p, plane=y, det=det)
    if kind == "stream":
        f, dms = _freqs(case["nchan"]), _dms(case)
        kinds = {
            "graded": (snd.Plan(f, dms, TSAMP_S, None, mode="graded", chunk=case["chunk"]), list(THRESHOLDS)),
            "float": (snd.Plan(f, dms, TSAMP_S, None, mode="float", in_dtype="bf16", node_dtype="bf16",
                               chunk=case["chunk"]), None),
        }
        server = Server(kinds, 64 << 30)
        names = {b: ("graded", "float")[b % 2] for b in range(case["beams"])}
        for b, k in names.items():
            assert server.admit(b, k)
        plan = kinds["graded"][0]
        n = -(-plan.max_delay // case["chunk"]) + 1  # chunks that a sweep spans: the sky repeats after them
        block = _filterbank(seed, case["nchan"], n * case["chunk"], case["dm_max"])
        chunks = [c.contiguous() for c in block.split(case["chunk"], dim=1)]
        s = dict(case=case, server=server, names=names, chunks=chunks)
        for _ in range(n):  # histories full, as in steady serving
            _push(s)
        return s
    if kind == "frontend":
        p = _power(case, seed)
        return dict(case=case, power=p, z=torch.empty_like(p))
    if kind == "multirate":
        mr = snd.MultiRate(_freqs(case["nchan"]), _dms(case), TSAMP_S, case["nsamp"], mode="graded", branching=8,
                           thresholds=THRESHOLDS, widths=WIDTHS_SCALED,
                           detect_kw=dict(n_base_widths=4, width_alpha=0.1, max_pixels=1 << 22))
        return dict(case=case, mr=mr, z=_filterbank(seed, case["nchan"], case["nsamp"], case["dm_max"]))
    f = snd.Fdmt(_freqs(case["nchan"]), BAND / case["nchan"], TSAMP_S, case["dm_max"], case["nsamp"])
    return dict(case=case, fdmt=f, x=_filterbank(seed, case["nchan"], case["nsamp"], case["dm_max"]),
                out=torch.empty((f.n_delays, case["nsamp"]), dtype=torch.float32, device="cuda"))


# ------------------------------------------------------------------------------- passes

def _table(cands):
    """Candidates as arrays of one size: whole numbers (DM row, time, width, cells) and S/N."""
    whole, snr = np.full((TABLE, 4), -1, dtype=np.int64), np.zeros(TABLE, dtype=np.float64)
    for i, c in enumerate(cands[:TABLE]):
        whole[i] = (c["k"], c["t"], c["width"], c["npix"])
        snr[i] = c["snr"]
    return dict(whole=whole, snr=snr)


def _push(s):
    server = s["server"]
    ready = []
    for b in server.beams():
        i = server.next_index(b)
        ready.append((b, i, s["chunks"][(i + b) % len(s["chunks"])]))
    return server.process(ready)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "tree":
        p, z = s["plan"], s["z"]
        if case["mode"] == "f32":
            x = z
        elif case["mode"] in ("bf16", "f16"):
            x = snd.cast(z, case["mode"])
        elif case["mode"] == "graded":
            x = snd.encode(z, THRESHOLDS, time_major=case["time_major"])
        elif p.in_dtype == "bits":
            x = snd.encode_bits(z, 2.0, time_major=case["time_major"])
        else:
            x = snd.encode(z, (2.0,), time_major=case["time_major"])
        y = p.execute(x, out=s["out"])
        if not case["detect"]:
            return dict(plane=y)
        return dict(plane=y, found=_table(s["det"].run(y)))
    if kind == "detect":
        found = _table(s["det"].run(s["plane"]))
        mu, sigma = s["det"].row_stats()
        return dict(found=found, mu=mu, sigma=sigma)
    if kind == "stream":
        res = _push(s)
        # a graded beam's candidates are whole numbers of its plane; a float beam's plane carries them
        return {str(b): dict(plane=s["server"].out[b], **({"found": _table(c)} if s["names"][b] == "graded" else {}))
                for b, _, _, _, c in res}
    if kind == "frontend":
        stats = snd.channel_stats(s["power"])
        z = snd.normalize(s["power"], stats, out=s["z"])
        flags, sigma = snd.flag_channels(z, case["window"], return_sigma=True)
        snd.zero_dm(z)
        return dict(stats=stats, flags=flags, sigma=sigma, z=z, bits=snd.encode_bits(z, 2.0))
    if kind == "multirate":
        merged, _ = s["mr"].run(s["z"])
        return dict(found=_table(merged))
    return dict(out=s["fdmt"].execute(s["x"], out=s["out"]))


# ------------------------------------------------------------------------------- work

def work(case):
    """Inputs read once, outputs written once; additions of a tree whose leaves are shared and whose
    upper levels are formed for each DM (a quarter of the channels per output sample)."""
    kind = case["kind"]
    if kind == "detect":
        nw = len(WIDTHS_SCALED if case["scaled"] else WIDTHS)
        cells = case["ndm"] * case["n_out"]
        return dict(bytes=4 * cells, flops=2 * nw * cells)
    if kind == "frontend":
        cells = case["nchan"] * case["nsamp"]
        return dict(bytes=8 * cells + cells / 8, flops=16 * cells)
    if kind == "fdmt":
        f = _freqs(case["nchan"])
        bw = BAND / case["nchan"]
        rows = math.ceil(KDM_MS * case["dm_max"] * ((f[-1] - bw / 2) ** -2 - (f[0] + bw / 2) ** -2) / (TSAMP_S * 1e3)) + 1
        return dict(bytes=4 * case["nsamp"] * (case["nchan"] + rows),
                    flops=rows * case["nsamp"] * math.log2(case["nchan"]))
    if kind == "stream":
        cells = case["ndm"] * case["chunk"]
        even, odd = (case["beams"] + 1) // 2, case["beams"] // 2
        return dict(bytes=case["beams"] * 4 * case["nchan"] * case["chunk"] + even * cells + odd * 4 * cells,
                    flops=case["beams"] * cells * case["nchan"] / 4)
    delay = int(_delays(_freqs(case["nchan"]), np.array([case["dm_max"]])).max())
    cells = case["ndm"] * (case["nsamp"] - delay)
    read = 4 * case["nchan"] * case["nsamp"]
    if kind == "multirate":
        return dict(bytes=read, flops=cells * case["nchan"] / 4 / 3)
    item = 4 if case["mode"] in ("f32", "bf16", "f16") else 1
    return dict(bytes=read + item * cells, flops=cells * case["nchan"] / 4 / (32 if case["mode"] == "bits" else 1))


# ------------------------------------------------------------------------------- in 64 bits

def _exact_plane(z, freqs, dms, n_out):
    """y[k][t] = sum over the channels of z[c][t + delay[k][c]], in float64 (some rows at a time)."""
    d = torch.from_numpy(_delays(freqs, dms)).cuda()
    z = z.double()
    y = torch.zeros((len(dms), n_out), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 28) // n_out)
    for k0 in range(0, len(dms), step):
        part = y[k0:k0 + step]
        for c in range(z.shape[0]):
            part += z[c].unfold(0, n_out, 1)[d[k0:k0 + step, c]]
    return y


def _exact_fdmt(case, x):
    """The transform's own recursion: halves of a band merged at the delays that split it by f^-2."""
    nchan, n = case["nchan"], case["nsamp"]
    f, bw = _freqs(nchan), BAND / nchan
    lo, hi = (lambda c: f[c] - 0.5 * bw), (lambda c: f[c] + 0.5 * bw)
    inv2 = lambda v: 1.0 / (v * v)  # noqa: E731
    band = inv2(lo(nchan - 1)) - inv2(hi(0))
    top = math.ceil(KDM_MS * case["dm_max"] * band / (TSAMP_S * 1e3))

    def count(c0, w):
        return min(top + 1, math.ceil(top * (inv2(lo(c0 + w - 1)) - inv2(hi(c0))) / band) + 1)

    x = x.double()
    rows = [x[c:c + 1].expand(count(c, 1), n) for c in range(nchan)]
    w = 2
    while w <= nchan:
        h, nxt = w // 2, []
        for s in range(nchan // w):
            up, low = rows[2 * s], rows[2 * s + 1]
            c0 = s * w
            split = (inv2(lo(c0 + h - 1)) - inv2(hi(c0))), (inv2(lo(c0 + w - 1)) - inv2(hi(c0)))
            m = count(c0, w)
            delta = np.arange(m)
            du = np.minimum(np.rint(delta * split[0] / split[1]).astype(np.int64), up.shape[0] - 1)
            dl = np.minimum(delta - du, low.shape[0] - 1)
            out = up[torch.from_numpy(du).cuda()]
            for i in range(m):
                if du[i] < n:
                    out[i, :n - du[i]] += low[dl[i], du[i]:]
            nxt.append(out)
        rows, w = nxt, 2 * w
    return rows[0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "tree" and case["mode"] in ("f32", "bf16", "f16"):
        f, dms = _freqs(case["nchan"]), _dms(case)
        z = _filterbank(seed, case["nchan"], case["nsamp"], case["dm_max"])
        return dict(plane=_exact_plane(z, f, dms, case["nsamp"] - int(_delays(f, dms).max())))
    if kind == "detect":
        y = prepare(case, seed)["plane"].double()
        mu = y.mean(dim=1)
        if case["sigma"] == "std":
            sigma = (y - mu[:, None]).square().mean(dim=1).sqrt()
        else:  # lower medians; the deviation is a float32 difference, as the plane's samples are
            y = y.float()
            m = y.median(dim=1, keepdim=True).values
            sigma = (y - m).abs().median(dim=1).values.double() * 1.4826022185056018
        return dict(found=None, mu=mu, sigma=sigma)
    if kind == "frontend":
        p = _power(case, seed).double()
        mu, sd = p.mean(dim=1, keepdim=True), p.std(dim=1, correction=0, keepdim=True)
        v = torch.minimum(torch.maximum(p, mu - 5.0 * sd), mu + 5.0 * sd)
        mu, sd = v.mean(dim=1, keepdim=True), v.std(dim=1, correction=0, keepdim=True)
        z = ((p - mu) / sd).float().double()
        w, sig = case["window"], []
        for a in range(0, case["nsamp"], w):
            part = z[:, a:a + w]
            s = part.std(dim=1, correction=0)
            m = s.median()
            dev = (s - m).abs()
            part[dev > 5.0 * (1.4826022185056018 * dev.median())] = 0.0
            sig.append(s)
        total = z.sum(dim=0)
        hit = total.abs() / math.sqrt(case["nchan"]) > 5.0
        z[:, hit] -= total[hit] / case["nchan"]
        return dict(stats=torch.cat([mu, sd], dim=1), flags=None, sigma=torch.stack(sig), z=z, bits=None)
    if kind == "fdmt":
        return dict(out=_exact_fdmt(case, _filterbank(seed, case["nchan"], case["nsamp"], case["dm_max"])))
    return None
