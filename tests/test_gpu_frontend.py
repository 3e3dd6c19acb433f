"""GPU parity of the front end (two-pass sigma-clip normalisation of raw power, then the
encoders) against the oracle."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def snd():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_2606_15361_amd as m
    return m


def test_sigma_clip_normalise_and_encode(snd, orc):
    rng = synth.make_rng(31)
    nchan, n = 96, 20000
    # raw power: chi-squared-like (exponential) with per-channel gains and offsets, RFI spikes
    p = (rng.exponential(1.0, (nchan, n)) * rng.uniform(0.5, 3.0, (nchan, 1)) + rng.uniform(0, 10, (nchan, 1)))
    p[5, 100:120] += 500.0
    p[17, ::997] += 80.0
    p[40] = 2.5  # a constant channel: sigma 0
    p[40, 7] = 2.5
    p = p.astype(np.float32)
    want_st = orc.sigma_clip_stats(p, 5.0)
    pt = torch.from_numpy(p).cuda()
    st = snd.channel_stats(pt, 5.0)
    got_st = st.cpu().numpy()
    ok = np.arange(nchan) != 40
    assert np.allclose(got_st[ok], want_st[ok], rtol=1e-12, atol=0.0)
    assert got_st[40, 0] == pytest.approx(2.5) and got_st[40, 1] == 0.0
    # normalise and encode the channels with sigma > 0 from the oracle's statistics: the
    # rasters must agree bit for bit (the same FP64 quotient, the same FP32 comparisons)
    sel = torch.from_numpy(np.flatnonzero(ok)).cuda()
    z = snd.normalize(pt[sel].contiguous(), torch.from_numpy(want_st[ok]).cuda())
    zw = orc.normalize(p[ok], want_st[ok])
    assert np.array_equal(z.cpu().numpy(), zw)
    for thr in ([1.5], [0.75], [1.0, 2.0, 3.0, 4.0]):
        assert np.array_equal(snd.encode(z, thr).cpu().numpy(), orc.encode(zw, thr))
    # with the GPU's own statistics the normalised values agree to FP64 rounding
    z2 = snd.normalize(pt[sel].contiguous(), st[sel].contiguous()).cpu().numpy()
    assert np.max(np.abs(z2 - zw)) <= 1e-5


def _flag_threshold_margin(sig, k):
    """Per window: distance of each channel's |s_c - m| from the flagging threshold
    k * MAD_SCALE * MAD, relative to the threshold (from the oracle's sigmas)."""
    import oracle
    out = np.empty_like(sig)
    for b in range(sig.shape[0]):
        s = sig[b]
        m = np.sort(s)[(s.size - 1) // 2]
        d = np.abs(s - m)
        thr = k * oracle.MAD_SCALE * np.sort(d)[(d.size - 1) // 2]
        out[b] = np.abs(d - thr) / max(thr, np.finfo(np.float64).tiny)
    return out


@pytest.mark.parametrize("nchan,n,window", [(96, 20011, 4096), (1024, 16384, 8192), (7, 1000, 1000)])
def test_flagging_and_zero_dm(snd, orc, nchan, n, window):
    # windowed MAD channel flagging, then zero-DM subtraction, on a z-scored block with RFI.
    # The oracle sums each window in time order, the kernel in its own order: the channel
    # sigmas agree to FP64 rounding (1e-12 relative).  A flag can then differ only for a channel
    # within that rounding of the threshold; no channel of this data comes within 1e-9 of it,
    # so the flags, and with them the zeroed samples, must agree exactly.  Zero-DM subtraction
    # then sums each sample's channels in channel order on both sides: bit-exact.
    rng = synth.make_rng(nchan + window)
    z = rng.standard_normal((nchan, n)).astype(np.float32)
    z[nchan // 3, : min(n, window)] *= 12.0            # hot channel in the first window
    z[nchan // 2, :] = 0.0                              # dead channel
    z[:, n // 2] += 8.0 / np.sqrt(nchan) * 3.0          # broadband spikes (zero-DM S/N ~ 24)
    z[:, n // 3: n // 3 + 5] += 2.0
    z[1, 17] += 40.0                                    # narrow-band spike
    zt = torch.from_numpy(z).cuda()
    flags, sig = snd.flag_channels(zt, window, k=5.0, return_sigma=True)
    want_z, want_f, want_s = orc.flag_channels(z, window, k=5.0, return_sigma=True)
    got_s = sig.cpu().numpy()
    assert np.allclose(got_s, want_s, rtol=1e-12, atol=1e-300)
    assert np.all((got_s == 0) == (want_s == 0))        # the dead channel is exactly 0 on both sides
    assert np.all(_flag_threshold_margin(want_s, 5.0) > 1e-9), "a channel sits on the flag threshold"
    assert np.array_equal(flags.cpu().numpy(), want_f)
    assert np.array_equal(zt.cpu().numpy(), want_z)
    assert want_f[0, nchan // 3] == 1 and np.all(want_f[:, nchan // 2] == 1)
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    snd.zero_dm(zt, 5.0, count=cnt)
    want_z2, want_n = orc.zero_dm(want_z, 5.0)
    assert int(cnt.item()) == want_n and want_n >= 1  # at least the strong broadband spike
    assert np.array_equal(zt.cpu().numpy(), want_z2)


@pytest.mark.parametrize("nchan,n", [(3, 1), (5, 67), (64, 255), (65, 1025), (70, 4096), (2, 4097), (130, 8195)])
def test_row_ends_and_unaligned_rows(snd, orc, nchan, n):
    """Encoders in both orders, casts, scrunch, normalisation and zero-DM at row lengths around a
    workgroup's samples and channel counts around a 64-channel tile, on rows that start on any element
    (a column offset into a wider block): the oracle's results, and no write past a row's end."""
    rng = synth.make_rng(nchan * 10007 + n)
    wide = rng.standard_normal((nchan, n + 5)).astype(np.float32)
    wide[0, n // 2] = np.nan
    block = torch.from_numpy(wide).cuda()
    for off in (0, 1, 3):
        z = wide[:, off:off + n]
        zt = block[:, off:off + n]
        th = [-0.5, 0.25, 1.0]
        want = orc.encode(z, th)
        for tm in (False, True):
            guard = torch.full((nchan, n + 7), 77, dtype=torch.uint8, device="cuda")
            src = block.t().contiguous()[off:off + n] if tm else zt
            snd.encode(src, th, time_major=tm, out=guard[:, 2:2 + n])
            g = guard.cpu().numpy()
            assert np.array_equal(g[:, 2:2 + n], want) and np.all(g[:, :2] == 77) and np.all(g[:, 2 + n:] == 77)
            words = torch.full((nchan, (n + 31) // 32 + 2), -1, dtype=torch.int32, device="cuda")
            snd.encode_bits(src, 0.25, time_major=tm, out=words)
            bits = np.unpackbits(words.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
            assert np.array_equal(bits[:, :n], orc.encode(z, [0.25]))
            pad = (n + 31) // 32 * 32
            assert np.all(bits[:, n:pad] == 0) and np.all(bits[:, pad:] == 1)
        fin = np.nan_to_num(z)
        ft = torch.nan_to_num(zt)
        for dt, tt in (("bf16", torch.bfloat16), ("f16", torch.float16)):
            assert torch.equal(snd.cast(zt, dt).cpu()[1:], torch.from_numpy(z[1:].copy()).to(tt))
        for s in (1, 2, 3, 4, 8, 16):
            if n // s:
                assert np.array_equal(snd.scrunch(zt, s).cpu().numpy()[1:], orc.scrunch(z, s)[1:])
        st = np.stack([fin.mean(1, dtype=np.float64), np.full(nchan, 1.5)], axis=1)
        assert np.array_equal(snd.normalize(zt, torch.from_numpy(st).cuda()).cpu().numpy()[1:], orc.normalize(z, st)[1:])
        for gamma in (1.0, 0.0):  # some samples of a wave corrected, then all of them
            y = ft.clone()
            snd.zero_dm(y, gamma)
            assert np.array_equal(y.cpu().numpy(), orc.zero_dm(fin, gamma)[0])


@pytest.mark.parametrize("nchan,n,window", [(5, 1000, 1), (130, 700, 63), (9, 1300, 64), (64, 2000, 100), (1100, 900, 257),
                                            (3, 4099, 512), (66, 5000, 513), (5, 9000, 2048), (6, 20000, 2049),
                                            (3, 17000, 8191), (65, 16384, 8192), (3, 30000, 8193), (2, 70001, 30000)])
def test_flagging_sums_in_the_stated_order(snd, orc, nchan, n, window):
    """The window sigmas are those of 64 interleaved FP64 partial sums, partial j over samples j, j + 64, ...
    in order, added in order of j, to the last bit: windows shorter and longer than a wave, around the sizes
    a wave holds in registers and past them, on rows that start on any element; and the oracle's flags."""
    z = synth.make_rng(nchan + n + window).standard_normal((nchan, n + 1)).astype(np.float32) * 3.0
    z[0, n // 2] = 1e6
    z = z[:, 1:]
    block = torch.zeros((nchan, n + 3), device="cuda")
    zt = block[:, 1:1 + n]
    zt.copy_(torch.from_numpy(z))
    flags, sig = snd.flag_channels(zt, window, k=4.0, return_sigma=True)

    def ordered(v):  # [nchan][samples] float64
        part = np.zeros((nchan, 64))
        for i in range(0, v.shape[1], 64):
            part[:, :v[:, i:i + 64].shape[1]] += v[:, i:i + 64]
        s = np.zeros(nchan)
        for j in range(64):
            s = s + part[:, j]
        return s

    got = sig.cpu().numpy()
    for b in range(got.shape[0]):
        x = z[:, b * window:(b + 1) * window].astype(np.float64)
        d = x - (ordered(x) / x.shape[1])[:, None]
        assert np.array_equal(got[b], np.sqrt(ordered(d * d) / x.shape[1])), b
    want_z, want_f = orc.flag_channels(np.ascontiguousarray(z), window, k=4.0)
    ok = np.all(_flag_threshold_margin(got, 4.0) > 1e-9, axis=1)  # windows with no channel on the threshold
    assert np.array_equal(flags.cpu().numpy()[ok], want_f[ok])
    y = zt.cpu().numpy()
    for b in np.flatnonzero(ok):
        assert np.array_equal(y[:, b * window:(b + 1) * window], want_z[:, b * window:(b + 1) * window])
    assert not block[:, 0].any() and not block[:, 1 + n:].any()


@pytest.mark.parametrize("nchan,n,window", [(300, 3000, 10), (257, 2001, 20), (40, 700, 5), (1000, 5003, 39), (5, 60, 20)])
def test_flagging_many_short_windows(snd, orc, nchan, n, window):
    """Windows that share their channels among several workgroups or take one each, with hot and dead
    channels at the ends of the shares: the oracle's flags and zeroed samples."""
    z = synth.make_rng(nchan * n + window).standard_normal((nchan, n)).astype(np.float32)
    z[0] *= 40.0
    z[-1] = 0.0
    z[nchan // 2, : n // 2] *= 25.0
    zt = torch.from_numpy(z).cuda()
    flags = snd.flag_channels(zt, window, k=6.0).cpu().numpy()
    want_z, want_f, sig = orc.flag_channels(z, window, k=6.0, return_sigma=True)
    ok = np.all(_flag_threshold_margin(sig, 6.0) > 1e-9, axis=1)
    assert ok.any() and want_f[ok].any()
    assert np.array_equal(flags[ok], want_f[ok])
    y = zt.cpu().numpy()
    for b in np.flatnonzero(ok):
        assert np.array_equal(y[:, b * window:(b + 1) * window], want_z[:, b * window:(b + 1) * window])


@pytest.mark.parametrize("n", [1, 3, 63, 257, 1023, 1024, 1025, 4099, 16384, 16385, 33001])
def test_channel_stats_by_row_length(snd, orc, n):
    """Clipped statistics of rows around each workgroup size, on rows that start on any element, with
    bright samples that the clip moves, a constant and a NaN row: the oracle's to FP64 rounding."""
    rng = synth.make_rng(n)
    p = (rng.standard_normal((7, n + 1)) * 3.0 + 100.0).astype(np.float32)
    p[2, n // 2] = 5000.0
    p[3] = 17.25
    p[6, n // 3 + 1] = np.nan
    x = p[:, 1:]
    block = torch.zeros((7, n + 2), device="cuda")
    xt = block[:, 1:1 + n]
    xt.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    got = snd.channel_stats(xt, clip=5.0).cpu().numpy()
    want = orc.sigma_clip_stats(np.ascontiguousarray(x[:6]), 5.0)
    # (the variance is E[d^2] - E[d]^2 about a sample of the row: rounding of its ten-fold squares)
    assert np.allclose(got[:6, 0], want[:, 0], rtol=1e-12, atol=0)
    assert np.allclose(got[:6, 1], want[:, 1], rtol=1e-9, atol=1e-9)
    assert got[3, 1] == 0.0 and np.isnan(got[6, 0])


@pytest.mark.parametrize("nchan,n", [(1000, 32805), (130, 90001), (70, 5000), (2, 129), (64, 256), (129, 1023)])
def test_time_major_tiles(snd, orc, nchan, n):
    """Both tile lengths of the time-major encoders (the longer ones in blocks that fill the chip), with
    ragged ends in channels and time, infinities and NaNs: the oracle's levels and bits, the channel-major
    encoders' too, and nothing written past a row."""
    z = synth.make_rng(nchan + n).standard_normal((nchan, n)).astype(np.float32)
    z[0, :: 7], z[-1, 1:: 11], z[nchan // 2, n - 1] = np.inf, np.nan, -np.inf
    th = [-0.5, 0.25, 1.0]
    want, want1 = orc.encode(z, th), orc.encode(z, [0.25])
    zt = torch.from_numpy(z).cuda()
    for tm in (True, False):
        src = zt.t().contiguous() if tm else zt
        guard = torch.full((nchan, n + 7), 77, dtype=torch.uint8, device="cuda")
        snd.encode(src, th, time_major=tm, out=guard[:, 3:3 + n])
        g = guard.cpu().numpy()
        assert np.array_equal(g[:, 3:3 + n], want) and np.all(g[:, :3] == 77) and np.all(g[:, 3 + n:] == 77)
        words = torch.full((nchan, (n + 31) // 32 + 2), -1, dtype=torch.int32, device="cuda")
        snd.encode_bits(src, 0.25, time_major=tm, out=words)
        bits = np.unpackbits(words.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
        pad = (n + 31) // 32 * 32
        assert np.array_equal(bits[:, :n], want1) and np.all(bits[:, n:pad] == 0) and np.all(bits[:, pad:] == 1)


@pytest.mark.parametrize("n", [97, 4096, 5003])
def test_non_finite_samples(snd, orc, n):
    """NaNs and infinities through the casts, the scrunch, the normalisation and zero-DM subtraction (a NaN
    never exceeds gamma, an infinite sum does): the oracle's values, NaNs where it has them."""
    rng = synth.make_rng(n)
    z = rng.standard_normal((9, n)).astype(np.float32)
    z[0, n // 2], z[1, 3], z[2, n - 1], z[8, :: 5] = np.nan, np.inf, -np.inf, np.nan
    zt = torch.from_numpy(z).cuda()
    for dt, tt in (("bf16", torch.bfloat16), ("f16", torch.float16)):
        got, want = snd.cast(zt, dt).cpu().float().numpy(), torch.from_numpy(z).to(tt).float().numpy()
        assert np.array_equal(got, want, equal_nan=True)
    st = np.stack([np.linspace(-1.0, 1.0, 9), np.linspace(0.5, 2.0, 9)], axis=1)
    with np.errstate(invalid="ignore"):
        for s in (1, 2, 4, 5, 8, 16):
            assert np.array_equal(snd.scrunch(zt, s).cpu().numpy(), orc.scrunch(z, s), equal_nan=True)
        assert np.array_equal(snd.normalize(zt, torch.from_numpy(st).cuda()).cpu().numpy(), orc.normalize(z, st),
                              equal_nan=True)
        y = zt.clone()
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        snd.zero_dm(y, 1.5, count=cnt)
        want, hits = orc.zero_dm(z, 1.5)
    assert np.array_equal(y.cpu().numpy(), want, equal_nan=True) and int(cnt.item()) == hits
