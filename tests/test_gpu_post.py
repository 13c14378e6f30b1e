"""Post-integration reductions on the GPU against the FP64 oracle (oracle/post.py), through the C ABI: channel
averaging with flags (Sec. 4), the smoothed bandpass and bandpass variation (Sec. 3.3.2), band moments and the
Allan variances of Eq. 3 and Eq. 4 (Sec. 3.3.1, 3.3.3).

Inputs are FP32 spectra (the library's Stokes output format); both sides compute in FP64.  Bounds: counts
bit-exact; FP32 outputs within 1e-6 relative of the oracle (one rounding to FP32 plus FP64 summation-order
differences); FP64 outputs (moments, Allan variances) within 1e-10 relative.
"""
import sys

import warnings

import numpy as np
import pytest

from oracle import post

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_1412_1256_amd as pk
    pk.lib()
    return torch, pk, torch.device("cuda:0")


def rel_close(got, ref, rtol):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    m = ~np.isnan(ref)
    err = np.max(np.abs(got[m] - ref[m]) / np.maximum(np.abs(ref[m]), 1e-30)) if m.any() else 0.0
    assert err <= rtol, err
    return err


def spectra(n_spec, C, seed, nan_edges=0):
    rng = np.random.default_rng(seed)
    k = np.arange(C)
    x = (1 + 0.2 * np.sin(k / 5000.0))[None] * (1 + 0.01 * rng.standard_normal((n_spec, C)))
    x = x.astype(np.float32)
    if nan_edges:
        x[:, :nan_edges] = np.nan
        x[:, C - nan_edges:] = np.nan
    return x


@pytest.mark.parametrize("factor", [1, 16, 32, 96, 256, 4096, 8192])
def test_channel_average_with_flags(env, factor):
    torch, pk, dev = env
    C = 131072 if factor != 96 else 96 * 1000
    say(f"channel average factor={factor} C={C}")
    x = spectra(8, C, factor, nan_edges=100)
    flags = np.zeros(C, dtype=np.uint8)
    flags[[5, 777, C // 2, C // 2 + 1, C - 300]] = 1
    x[:, C // 2] = 1e9  # a spurious channel (flagged)
    out, cnt = pk.channel_average(torch.from_numpy(x).to(dev), factor, torch.from_numpy(flags).to(dev))
    torch.cuda.synchronize(dev)
    ref, rcnt = post.channel_average(x, factor, flags)
    assert np.array_equal(cnt.cpu().numpy(), rcnt)
    e = rel_close(out.cpu().numpy(), ref, 1e-6)
    say(f"  err {e}")


def test_channel_average_of_stokes_output(env):
    """The paper's TMC-1 reduction on the library's own Stokes output: 131072 channels to 4096 (1.95 kHz)."""
    torch, pk, dev = env
    import synth
    inst = synth.make_paper(n_frames=8)
    plan = pk.Plan([pk.Instance.from_synth(inst)], device=dev)
    plan.reset()
    plan.accumulate(torch.from_numpy(inst["packed"]).to(dev))
    st = plan.stokes()
    flags = torch.zeros(st.shape[-1], dtype=torch.uint8, device=dev)
    flags[65536] = 1
    out, cnt = pk.channel_average(st, 32, flags)
    torch.cuda.synchronize(dev)
    assert out.shape == (1, 4, 4096)
    ref, rcnt = post.channel_average(st.cpu().numpy().reshape(4, -1), 32, flags.cpu().numpy())
    assert np.array_equal(cnt.cpu().numpy().reshape(4, -1), rcnt)
    rel_close(out.cpu().numpy().reshape(4, -1), ref, 1e-6)


@pytest.mark.parametrize("C,K,edge", [(131072, 128, 0.06), (8192, 128, 0.06), (5000, 96, 0.1), (1 << 20, 512, 0.06),
                                      (4096, 64, 0.0)])
def test_bandpass_fit(env, C, K, edge):
    torch, pk, dev = env
    say(f"bandpass fit C={C} K={K} edge={edge}")
    rng = np.random.default_rng(C + K)
    k = np.arange(C)
    h = (1 + 0.3 * np.sin(k / (C / 7.0)) + 0.05 * np.cos(k / 311.0) + 0.01 * rng.standard_normal(C)).astype(np.float32)
    got = pk.bandpass_fit(torch.from_numpy(h).to(dev), K, edge).cpu().numpy()
    ref, _ = post.bandpass_fit(h, K, edge)
    e = rel_close(got, ref, 1e-6)
    say(f"  err {e}")


@pytest.mark.parametrize("n_int,rest", [(4, 0), (5, 7), (6, 0), (60, 9), (92, 3), (93, 0), (1021, 0), (1533, 15),
                                        (3069, 0)])
def test_bandpass_solve_sizes(env, n_int, rest):
    """The banded solve at the edges of its blocking: n_int (+ 1 partial interval of `rest` channels) + 3
    coefficients in blocks of three, one to 1024 of them, partly filled, and around powers of two and whole waves.
    16-channel knots, no edges; FP32 output: half an ulp (6e-8) plus FP64 solve errors far below, bound 1e-6."""
    torch, pk, dev = env
    C = 16 * n_int + rest
    h = spectra(1, C, 17 + n_int)[0]
    say(f"solve of {n_int + (rest > 0) + 3} coefficients")
    got = pk.bandpass_fit(torch.from_numpy(h).to(dev), 16, 0.0).cpu().numpy()
    rel_close(got, post.bandpass_fit(h, 16, 0.0)[0], 1e-6)


def test_bandpass_correct_and_stats(env):
    torch, pk, dev = env
    C = 131072
    hk = spectra(30, C, 3)
    smooth = post.bandpass_fit(hk.mean(axis=0), 128, 0.06)[0].astype(np.float32)
    G = 1 + 0.01 * np.arange(30)
    got = pk.bandpass_correct(torch.from_numpy(hk).to(dev), torch.from_numpy(smooth).to(dev),
                              torch.from_numpy(G).to(dev))
    st = pk.band_stats(got)
    torch.cuda.synchronize(dev)
    ref = post.bandpass_correct(hk, smooth, G)
    rel_close(got.cpu().numpy(), ref, 1e-6)
    # moments of the GPU's own FP32 output
    rel_close(st.cpu().numpy(), post.band_stats(got.cpu().numpy()), 1e-10)


def test_bandpass_stability_chain(env):
    """Sec. 3.3.2 end to end: a series of integrations H_k with gain drift, the long-integration bandpass
    smoothed (128-channel knots, 6 % edges), H^_k = H_k / (G_k H), 256-channel averages, their mean and SD."""
    torch, pk, dev = env
    C, K = 131072, 30
    rng = np.random.default_rng(11)
    k = np.arange(C)
    shape = 1 + 0.4 * np.exp(-((k - C / 2) / (C / 3)) ** 2) + 0.02 * np.sin(k / 900.0)
    G = 1 + 0.002 * np.arange(K)
    hk = (G[:, None] * shape[None] * (1 + 2.6e-3 * rng.standard_normal((K, C)))).astype(np.float32)
    # GPU chain
    t_hk = torch.from_numpy(hk).to(dev)
    H = t_hk.double().mean(dim=0).float()
    smooth = pk.bandpass_fit(H, 128, 0.06)
    hat = pk.bandpass_correct(t_hk, smooth, torch.from_numpy(G).to(dev))
    binned, cnt = pk.channel_average(hat, 256)
    st = pk.band_stats(binned).cpu().numpy()
    torch.cuda.synchronize(dev)
    # oracle chain from the same FP32 series (its own FP64 arithmetic at every stage)
    sm_ref, _ = post.bandpass_fit(H.cpu().numpy(), 128, 0.06)
    hat_ref = post.bandpass_correct(hk, sm_ref, G)
    bin_ref, _ = post.channel_average(hat_ref, 256)
    st_ref = post.band_stats(bin_ref)
    say(f"  mean, SD of the first spectra {st[:3].tolist()}")
    assert np.max(np.abs(st[:, 0] - st_ref[:, 0])) < 1e-6
    assert np.max(np.abs(st[:, 1] / st_ref[:, 1] - 1)) < 1e-3
    # white noise of 2.6e-3 per channel, 256-channel bins: SD about 2.6e-3 / 16
    assert np.all(np.abs(st[:, 1] / (2.6e-3 / 16) - 1) < 0.3)


def test_time_allan_variance_across_channels(env):
    """TAV (Eq. 3) of every channel of a series of 1-s integrations, normalised by the mean."""
    torch, pk, dev = env
    T, C = 1200, 4096
    rng = np.random.default_rng(4)
    x = (1 + 0.001 * np.arange(T)[:, None] / T + 0.01 * rng.standard_normal((T, C))).astype(np.float32)
    lags = [1, 2, 4, 8, 16, 64, 256, 599, 600]
    got = pk.allan(torch.from_numpy(x).to(dev), lags, spacing=1.0, normalize=True, axis=0).cpu().numpy()
    ref = post.allan(x.T, lags, spacing=1.0, normalize=True)
    rel_close(got, ref, 1e-10)
    assert np.all(np.isnan(got[:, -1]))  # 2 L >= n_points


def test_time_allan_variance_window_form(env):
    """TAV of side-by-side series with every lag at most 512 (the LDS-window form): the benchmark's lag set over
    1800 1-s integrations, normalised, and a lag set of two groups with a non-multiple-of-32 channel count."""
    torch, pk, dev = env
    rng = np.random.default_rng(11)
    T, C = 1800, 2048
    x = (1 + 0.002 * np.sin(np.arange(T) / 97.0)[:, None] + 0.01 * rng.standard_normal((T, C))).astype(np.float32)
    lags = [1, 2, 4, 8, 16, 64, 256, 512]
    got = pk.allan(torch.from_numpy(x).to(dev), lags, spacing=1.0, normalize=True, axis=0).cpu().numpy()
    rel_close(got, post.allan(x.T, lags, spacing=1.0, normalize=True), 1e-10)
    # a partial last workgroup (998 series, the window form) and an odd series count (999, the column form),
    # infinite samples (left out), lags in two groups of eight, and lags with one or no term
    for C in (998, 999):
        T = 777
        x = (3 + 0.05 * rng.standard_normal((T, C))).astype(np.float32)
        x[rng.integers(0, T, 200), rng.integers(0, C, 200)] = np.inf
        lags = [1, 2, 3, 5, 8, 13, 21, 34, 55, 89, 144, 233, 377, 388, 389]
        got = pk.allan(torch.from_numpy(x).to(dev), lags, spacing=0.5, axis=0).cpu().numpy()
        ref = post.allan(x.T, lags, spacing=0.5)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        ok = ~np.isnan(ref)
        rel_close(got[ok], ref[ok], 1e-10)


def test_time_allan_variance_ragged_with_flags(env):
    """TAV of side-by-side series: a channel count that is not a whole number of 64-series workgroups, a
    series length that does not split evenly over the time slices, NaN (flagged) samples, both with and
    without normalisation; run twice, bitwise equal."""
    torch, pk, dev = env
    T, C = 1001, 1000
    rng = np.random.default_rng(9)
    x = (2 + 0.02 * rng.standard_normal((T, C))).astype(np.float32)
    x[rng.integers(0, T, 300), rng.integers(0, C, 300)] = np.nan
    x[:, 7] = np.nan  # a channel with no finite sample
    lags = [1, 3, 5, 17, 100, 250, 333, 499, 500, 501]
    xd = torch.from_numpy(x).to(dev)
    for normalize in (False, True):
        got = pk.allan(xd, lags, spacing=2.0, normalize=normalize, axis=0).cpu().numpy()
        again = pk.allan(xd, lags, spacing=2.0, normalize=normalize, axis=0).cpu().numpy()
        with warnings.catch_warnings():  # the mean of the all-NaN channel is NaN by design
            warnings.simplefilter("ignore", RuntimeWarning)
            ref = post.allan(x.T, lags, spacing=2.0, normalize=normalize)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        ok = ~np.isnan(ref)
        rel_close(got[ok], ref[ok], 1e-10)
        assert np.array_equal(np.nan_to_num(got), np.nan_to_num(again))
        assert np.all(np.isnan(got[7])) and np.all(np.isnan(got[:, -1]))


def test_spectral_allan_variance(env):
    """SAV (Eq. 4) along the channels of bandpass-corrected spectra with NaN band edges."""
    torch, pk, dev = env
    x = spectra(6, 131072, 8, nan_edges=7864)
    lags = [1, 2, 4, 16, 128, 1024]
    got = pk.allan(torch.from_numpy(x).to(dev), lags, spacing=61.03515625, axis=1).cpu().numpy()
    ref = post.allan(x, lags, spacing=61.03515625)
    rel_close(got, ref, 1e-10)
    # normalised, and a series length that is not a whole number of 4096-point chunks
    y = torch.from_numpy(x[:, :100000].copy()).to(dev)
    got = pk.allan(y, lags, spacing=61.03515625, normalize=True, axis=1).cpu().numpy()
    rel_close(got, post.allan(x[:, :100000], lags, spacing=61.03515625, normalize=True), 1e-10)


def test_post_reductions_are_deterministic(env):
    torch, pk, dev = env
    x = torch.from_numpy(spectra(4, 131072, 5)).to(dev)
    a = [pk.channel_average(x, 32)[0], pk.band_stats(x), pk.allan(x, [1, 8], axis=1), pk.bandpass_fit(x[0])]
    b = [pk.channel_average(x, 32)[0], pk.band_stats(x), pk.allan(x, [1, 8], axis=1), pk.bandpass_fit(x[0])]
    torch.cuda.synchronize(dev)
    for u, v in zip(a, b):
        assert torch.equal(torch.nan_to_num(u), torch.nan_to_num(v))


@pytest.mark.parametrize("n,bad", [(1, 0), (64, 0), (1024, 3), (1026, 0), (4096, 0), (4097, 1), (4608, 0), (12289, 2),
                                   (28672, 0), (28673, 4), (40000, 700)])
def test_allan_consecutive_points(env, n, bad):
    """Series of consecutive points around the edges of the 4096-point chunks and the longest staged lag (512), and
    past it (513), with non-finite samples; the chunk sums by a thread (under 8 chunks) and by a wave per lag.
    FP64 sums in another order: relative differences of order n eps, bound 1e-10."""
    torch, pk, dev = env
    rng = np.random.default_rng(n)
    x = (1 + 0.01 * rng.standard_normal((3, n))).astype(np.float32)
    if bad:
        x[1, rng.integers(0, n, bad)] = np.nan
        x[2, -bad:] = np.inf
    for lags in ([1, 2, 3, 31, 64, 255, 511, 512, 5], [513, 7]):
        say(f"allan n={n} bad={bad} lags={lags}")
        for norm in (False, True):
            with warnings.catch_warnings():
                warnings.simplefilter("ignore")
                ref = post.allan(x, lags, 2.0, norm)
            got = pk.allan(torch.from_numpy(x).to(dev), lags, 2.0, normalize=norm, axis=1).cpu().numpy()
            rel_close(got, ref, 1e-10)


@pytest.mark.parametrize("factor,bins", [(63, 5), (64, 7), (65, 1), (255, 9), (256, 4), (257, 3), (2047, 2), (2048, 3),
                                         (2049, 2)])
def test_channel_average_factor_edges(env, factor, bins):
    """Bins around the changes of form (64 and 2048 channels) and of the wave's rounds of 256, and a count of bins
    that does not fill a workgroup; counts exact, means within one FP32 rounding (1e-6)."""
    torch, pk, dev = env
    x = spectra(3, factor * bins, factor, nan_edges=5)
    flags = (np.arange(factor * bins) % 11 == 3).astype(np.uint8)
    for fl in (None, flags):
        out, cnt = pk.channel_average(torch.from_numpy(x).to(dev), factor,
                                      None if fl is None else torch.from_numpy(fl).to(dev))
        ref, rcnt = post.channel_average(x, factor, fl)
        assert np.array_equal(cnt.cpu().numpy(), rcnt)
        rel_close(out.cpu().numpy(), ref, 1e-6)


@pytest.mark.parametrize("n,shift", [(4, 0), (1020, 0), (1024, 1), (1028, 0), (1030, 0), (5000, 2)])
def test_bandpass_correct_alignment(env, n, shift):
    """Rows of whole aligned quadruples, and rows that are not (odd lengths, buffers that start off 16 bytes)."""
    torch, pk, dev = env
    hk, sm = spectra(3, n, n), spectra(1, n, n + 1)[0]
    G = np.array([1.0, 0.5, 3.0])
    t = torch.zeros(3 * n + 4, device=dev)[shift:shift + 3 * n].view(3, n)
    t.copy_(torch.from_numpy(hk))
    got = pk.bandpass_correct(t, torch.from_numpy(sm).to(dev), torch.from_numpy(G).to(dev))
    rel_close(got.cpu().numpy(), post.bandpass_correct(hk, sm, G), 1e-6)


@pytest.mark.parametrize("P,n", [(1, 64), (2, 66), (3, 65), (100, 68), (286, 129), (287, 132), (572, 70), (573, 96),
                                 (1144, 80), (1145, 67), (1800, 72), (2288, 64), (2289, 64)])
def test_allan_side_by_side_sizes(env, P, n):
    """Side-by-side series at the edges of the whole-series form's widths (8, 16, 32 and 64 series to a workgroup; past
    2288 points the window form), with whole and ragged groups of series, lags that cut runs evenly and not, lags
    without a term, and non-finite samples.  FP64 sums in another order: of order P eps, bound 1e-10."""
    torch, pk, dev = env
    rng = np.random.default_rng(P + n)
    x = (1 + 0.01 * rng.standard_normal((P, n))).astype(np.float32)
    lags = [1, 2, 3, 7, 33, 45, 64, 65, 127, 256, 500, max(1, (P - 1) // 2), P // 2 + 1, 2 ** 31 - 1]
    for bad in (False, True):
        if bad:
            x[P // 2, 1] = np.nan
            x[0, n - 1] = np.inf
            x[:, 5] = -np.inf
            x[P // 3, 6] = 3e38
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            ref = post.allan(x.T, lags, 0.5, bad)
        say(f"allan side by side P={P} n={n} bad={bad}")
        got = pk.allan(torch.from_numpy(x).to(dev), lags, 0.5, normalize=bad, axis=0).cpu().numpy()
        rel_close(got, ref, 1e-10)


@pytest.mark.parametrize("K,n_int,rest", [(1024, 4, 2), (1025, 4, 1000), (4096, 5, 2), (8191, 4, 300), (8192, 4, 0),
                                          (8192, 4, 1025), (20000, 6, 777)])
def test_bandpass_wide_knots(env, K, n_int, rest):
    """Intervals of one, four and sixteen waves, with partial last intervals shorter than their lanes; NaN-free spectra,
    FP32 output: half an ulp (6e-8) plus FP64 errors far below, bound 1e-6."""
    torch, pk, dev = env
    C = K * n_int + rest
    h = spectra(1, C, 40 + K)[0]
    say(f"{n_int} intervals of {K} channels and {rest}")
    got = pk.bandpass_fit(torch.from_numpy(h).to(dev), K, 0.0).cpu().numpy()
    rel_close(got, post.bandpass_fit(h, K, 0.0)[0], 1e-6)


@pytest.mark.parametrize("n_lags", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("bad", [0, 3])
def test_allan_few_lags(env, n_lags, bad):
    """Series of consecutive points at as many lags as each kernel of a sweep serves, and one more; FP64 sums in another
    order: relative differences of order n eps, bound 1e-10."""
    torch, pk, dev = env
    rng = np.random.default_rng(n_lags)
    x = (1 + 0.01 * rng.standard_normal((4, 40001))).astype(np.float32)
    if bad:
        x[1, rng.integers(0, 40001, bad)] = np.nan
        x[3, :bad] = np.inf
    lags = [1, 512, 3, 77, 256, 5, 2, 300, 8][:n_lags]
    say(f"{n_lags} lags, bad={bad}")
    for norm in (False, True):
        ref = post.allan(x, lags, 2.0, norm)
        got = pk.allan(torch.from_numpy(x).to(dev), lags, 2.0, normalize=norm, axis=1).cpu().numpy()
        rel_close(got, ref, 1e-10)


@pytest.mark.parametrize("P,n", [(5, 16320), (5, 16321), (100, 16324), (286, 16385), (287, 8160), (287, 8161), (572, 8164),
                                 (573, 2032), (573, 2033), (1144, 2036), (1145, 2033)])
def test_allan_widths_of_many_series(env, P, n):
    """Enough side-by-side series for 64, 32 and 16 of them to a workgroup, and one group fewer; ragged last groups, odd
    counts and non-finite samples.  Second differences of FP32 samples are exact in FP64 (not so those of samples divided by
    their mean, hence not normalised); their sums in another order: of order P eps, bound 1e-10."""
    torch, pk, dev = env
    rng = np.random.default_rng(P + n)
    x = (1 + 0.01 * rng.standard_normal((P, n))).astype(np.float32)
    x[P // 2, 1] = np.nan
    x[0, n - 1] = np.inf
    x[:, n - 70] = -np.inf
    lags = [1, 2, 7, 33, 64, 127, max(1, (P - 1) // 2), P // 2 + 1]
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        ref = post.allan(x.T, lags, 0.5)
    say(f"allan side by side P={P} n={n}")
    got = pk.allan(torch.from_numpy(x).to(dev), lags, 0.5, axis=0).cpu().numpy()
    rel_close(got, ref, 1e-10)


@pytest.mark.parametrize("factor", [64, 65, 127, 128, 129])
@pytest.mark.parametrize("bins", [1, 2, 3, 5, 16, 17])
def test_channel_average_bins_of_a_wave(env, factor, bins):
    """Bins that waves take in fours, twos and singly, in numbers that leave the last wave's group and the last workgroup
    partly filled; flagged, non-finite and wholly flagged bins.  Counts exact, means within one FP32 rounding (1e-6)."""
    torch, pk, dev = env
    x = spectra(2, factor * bins, factor + bins)
    x[1, ::7] = np.inf
    flags = (np.arange(factor * bins) % 5 == 3).astype(np.uint8)
    flags[(bins - 1) * factor:] = 1
    for fl in (None, flags):
        out, cnt = pk.channel_average(torch.from_numpy(x).to(dev), factor,
                                      None if fl is None else torch.from_numpy(fl).to(dev))
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            ref, rcnt = post.channel_average(x, factor, fl)
        assert np.array_equal(cnt.cpu().numpy(), rcnt)
        rel_close(out.cpu().numpy(), ref, 1e-6)
