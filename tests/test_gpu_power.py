"""Level histograms and total power on the GPU (counted inside the column pass) against the oracle:
counts bit-exact, power estimates to FP64 rounding (both sides evaluate the same sums and erfinv)."""
import sys

import numpy as np
import pytest

import oracle
import synth

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


def run(env, d, calls=1, hist=True):
    torch, pk, dev = env
    plan = pk.Plan([pk.Instance.from_synth(d)], device=dev)
    if hist:
        plan.set_histograms(True)
    packed = torch.from_numpy(d["packed"]).to(dev)
    plan.reset()
    per = d["n_frames"] // calls * d["fft_len"] * d["n_streams"] * d["bits"] // 8
    for c in range(calls):
        plan.accumulate(packed[c * per:packed.numel() if c == calls - 1 else (c + 1) * per])
    spec = plan.spectra()[0].cpu().numpy()
    if not hist:
        return spec, None, None, 0
    counts, power, nf = plan.histograms()
    return spec, counts.cpu().numpy(), power.cpu().numpy(), nf


@pytest.mark.parametrize("bits,log2n,F", [(2, 12, 9), (4, 14, 5), (8, 16, 6), (2, 18, 3), (8, 18, 3)])
def test_two_streams(env, bits, log2n, F):
    say(f"histograms bits={bits} N=2^{log2n} F={F}")
    d = synth.make_correlated_noise(bits, 0.3, 1 << log2n, F, seed_extra=log2n + bits)
    spec, counts, power, nf = run(env, d, calls=2 if F > 3 else 1)
    ref = oracle.level_histograms(d["packed"], bits, 2, d["n_samples"], d["pairs"])
    assert nf == F
    assert np.array_equal(counts, ref)
    pref = oracle.total_power(ref, bits)
    assert np.allclose(power[..., 0], pref[..., 0], rtol=1e-13, atol=0)
    if bits == 2:
        assert np.allclose(power[..., 1], pref[..., 1], rtol=1e-12, atol=0)
    else:
        assert np.all(np.isnan(power[..., 1]))
    # counting does not change the spectra: bitwise where both runs take the four-step passes; transforms of
    # 2^12 points or less run the single pass when not counting, equal within FP32 rounding
    spec_off = run(env, d, calls=2 if F > 3 else 1, hist=False)[0]
    if log2n > 12:
        assert np.array_equal(spec, spec_off)
    else:
        scale = np.mean(spec_off[:, 0:1, :], axis=2, keepdims=True)
        assert np.max(np.abs(spec - spec_off) / scale) < 2e-6


def test_four_streams_two_pairs(env):
    say("histograms 4 int8 streams, pairs (0,2), (1,3)")
    d = synth.make_precision(n_frames=2, fft_len=1 << 14)
    spec, counts, power, nf = run(env, d)
    ref = oracle.level_histograms(d["packed"], 8, 4, d["n_samples"], d["pairs"])
    assert np.array_equal(counts, ref)


def test_reset_and_errors(env):
    torch, pk, dev = env
    say("histogram state and errors")
    d = synth.make_correlated_noise(2, 0.1, 1 << 12, 4, seed_extra=77)
    plan = pk.Plan([pk.Instance.from_synth(d)], device=dev)
    packed = torch.from_numpy(d["packed"]).to(dev)
    with pytest.raises(pk.PolarisError) as e:
        plan.histograms()
    assert e.value.code == "PS_ERR_STATE"
    plan.set_histograms(True)
    plan.reset()
    plan.accumulate(packed)
    plan.accumulate(packed)
    c2 = plan.histograms()[0].cpu().numpy()
    plan.reset()
    plan.accumulate(packed)
    c1, _, nf = plan.histograms()
    assert nf == 4 and np.array_equal(2 * c1.cpu().numpy(), c2)
    with pytest.raises(pk.PolarisError) as e:
        plan.set_histograms(False)  # inside an integration
    assert e.value.code == "PS_ERR_STATE"
    f32 = pk.Plan([pk.Instance(fft_len=1 << 12, bits=32)], device=dev)
    with pytest.raises(pk.PolarisError) as e:
        f32.set_histograms(True)
    assert e.value.code == "PS_ERR_UNSUPPORTED"


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_histograms_read_separately(env, bits):
    """The counts alone, the estimates alone (the other pointer NULL) and both together are the same, for fewer bins
    than a wave has lanes and for more, with the streams of two pairs; whole numbers, so exact."""
    import ctypes as C
    torch, pk, dev = env
    rng = np.random.default_rng(bits)
    N, F = 1 << 13, 3
    packed = torch.from_numpy(rng.integers(0, 256, N * F * 4 * bits // 8, dtype=np.uint8)).to(dev)
    plan = pk.Plan([pk.Instance(fft_len=N, bits=bits, n_streams=4, pairs=((0, 2), (1, 3)))], device=dev)
    plan.set_histograms(True)
    plan.reset()
    plan.accumulate(packed)
    counts, power, _ = plan.histograms()
    only_c, only_p = torch.empty_like(counts), torch.empty_like(power)
    assert pk.lib().ps_histograms(plan._h, 0, C.c_void_p(only_c.data_ptr()), None, None) == 0
    assert pk.lib().ps_histograms(plan._h, 0, None, C.c_void_p(only_p.data_ptr()), None) == 0
    torch.cuda.synchronize(dev)
    assert torch.equal(only_c, counts) and torch.equal(only_p.nan_to_num(-1.0), power.nan_to_num(-1.0))
    assert int(counts.sum()) == 4 * N * F


@pytest.mark.parametrize("log2n,F,pairs", [(8, 1500, 1), (9, 40, 1), (10, 300, 1), (11, 70, 2), (12, 200, 1), (12, 600, 2)])
def test_slots_of_counted_integrations(env, log2n, F, pairs):
    """Integrations of short transforms with histograms use fewer accumulator slots than those without.  Spectra against
    the FP64 oracle (1e-5 of the mean power), split calls bitwise; a state exported with fewer slots in use resumes in a
    plan that uses all (FP64 sums in another order, 1e-12); a captured integration with histograms is read in its own
    slots after integrations without."""
    torch, pk, dev = env
    N = 1 << log2n
    say(f"N=2^{log2n} F={F} pairs={pairs}")
    d = synth.make_precision(n_frames=F, fft_len=N) if pairs == 2 else synth.make_correlated_noise(8, 0.3, N, F, seed_extra=5)
    inst = pk.Instance.from_synth(d, precision="fp32", accum="fp64")
    acc = oracle.run_instance(d)[0]
    packed = torch.from_numpy(d["packed"]).to(dev)
    per = N * d["n_streams"] * d["bits"] // 8
    cut = (F // 3) * per
    side = torch.cuda.Stream(dev)
    with torch.cuda.stream(side):
        counted = pk.Plan([inst], device=dev, stream=side)
        counted.set_histograms(True)

        def whole():
            counted.reset()
            counted.accumulate(packed)

        whole()
        got = counted.spectra()[0]
        assert np.max(np.abs(got.cpu().numpy() - acc)) < 1e-5 * acc[:, :2].mean()
        counted.reset()
        counted.accumulate(packed[:cut])
        state, n = counted.state_export()
        counted.accumulate(packed[cut:])
        assert torch.equal(counted.spectra()[0], got)
        plain = pk.Plan([inst], device=dev, stream=side)
        plain.state_import(state, n)
        counted.reset()
        counted.accumulate(packed[:cut])
        a, b = plain.spectra()[0], counted.spectra()[0]
        assert float((a - b).abs().max() / b[:, :2].mean()) < 1e-12
        plain.accumulate(packed[cut:])
        assert float((plain.spectra()[0] - got).abs().max() / got[:, :2].mean()) < 1e-5
        counted.graph_capture(whole)
        for k in range(3):
            counted.reset()
            counted.set_histograms(False)
            counted.accumulate(packed[:cut * (k % 2 + 1)])
            counted.stokes()
            counted.reset()
            counted.set_histograms(True)
            counted.graph_replay()
            assert torch.equal(counted.spectra()[0], got), k
    torch.cuda.synchronize(dev)
