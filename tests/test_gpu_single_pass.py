"""Single-pass short transforms (whole frames in LDS, N = 2^8 .. 2^12) on the GPU against the FP64 oracle and
against the four-step passes, through the C ABI.

Bounds as in the plain parity tests: per Stokes product max_k |P_gpu - P_ref| / I_ref,k <= 1e-5 (>= 32
frames); spectra normwise max_k |d| / mean_k XX_ref <= 1e-5.  Single pass vs four-step: the same
quantities within FP32 rounding of the two transforms (normwise 2e-6).  Split calls and repeated runs:
bitwise equal.
"""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-5


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_1412_1256_amd as pk
    pk.lib()
    return torch, pk, torch.device("cuda:0")


def stokes_err(got, ref):
    return np.max(np.abs(got - ref) / ref[:, 0:1, :], axis=2)


def spectra_err(got, ref):
    return np.max(np.abs(got - ref) / np.mean(ref[:, 0:1, :], axis=2, keepdims=True), axis=2)


def run(env, inst, sched=None, calls=1, psi=0.0):
    torch, pk, dev = env
    plan = pk.Plan([pk.Instance.from_synth(inst)], device=dev, schedules=None if sched is None else [sched])
    packed = torch.from_numpy(inst["packed"]).to(dev)
    N, S, b = inst["fft_len"], inst["n_streams"], inst["bits"]
    F = inst["n_samples"] // N
    per = max(1, F // calls)
    cuts = [min(F, c * per) for c in range(calls)] + [F]
    plan.reset()
    for c in range(calls):
        plan.accumulate(packed[cuts[c] * N * S * b // 8:cuts[c + 1] * N * S * b // 8])
    spec, nf = plan.spectra()
    st = plan.stokes(psi=psi)
    torch.cuda.synchronize(dev)
    return spec.cpu().numpy(), nf, st.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("log2n", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("bits,window", [(2, "rect"), (4, "hann"), (8, "hamming"), (32, "blackman")])
def test_single_pass_against_oracle(env, log2n, bits, window):
    torch, pk, dev = env
    inst = synth.make_correlated_noise(bits, 0.3, 1 << log2n, 40, seed_extra=log2n * 10 + bits, window=window)
    say(f"single pass N=2^{log2n} bits={bits} {window}")
    acc, nf, s2, _ = oracle.run_instance(inst)
    ref = oracle.stokes(acc, nf, s2, psi=0.2)
    spec, gnf, st = run(env, inst, psi=0.2)
    assert gnf == nf == 40
    es, e = spectra_err(spec, acc), stokes_err(st, ref)
    say(f"  spectra {es.max()} stokes {e.tolist()}")
    assert np.all(es < TOL) and np.all(e < TOL)


@pytest.mark.parametrize("bits", [2, 8])
def test_four_streams_two_pairs(env, bits):
    torch, pk, dev = env
    rng = synth.rng_for(300, bits)
    N, F = 4096, 36
    base = rng.standard_normal((4, N * F))
    x = np.stack([base[0], base[1], 0.6 * base[0] + 0.8 * base[2], 0.3 * base[1] + 0.95 * base[3]], axis=1)
    if bits == 8:
        x = x * 16
    inst = dict(packed=synth.pack_codes(synth.quantize(x, bits), bits), bits=bits, n_streams=4, fft_len=N,
                n_frames=F, n_samples=N * F, window="rect", pairs=[(0, 2), (1, 3)])
    say(f"single pass four streams bits={bits}")
    acc, nf, s2, _ = oracle.run_instance(inst)
    ref = oracle.stokes(acc, nf, s2)
    spec, gnf, st = run(env, inst)
    assert np.all(stokes_err(st, ref) < TOL)


@pytest.mark.parametrize("log2n", [8, 10, 12])
def test_single_pass_matches_four_step(env, log2n):
    torch, pk, dev = env
    inst = synth.make_correlated_noise(8, 0.3, 1 << log2n, 64, seed_extra=log2n, window="hann")
    say(f"single pass vs four-step N=2^{log2n}")
    a, _, _ = run(env, inst)
    b, _, _ = run(env, inst, sched=pk.Schedule(single_pass=2))
    e = spectra_err(a, b)
    say(f"  {e.max()}")
    assert e.max() < 2e-6


@pytest.mark.parametrize("slots", [1, 4, 64, 1024])
def test_slot_counts_and_split_calls(env, slots):
    torch, pk, dev = env
    inst = synth.make_correlated_noise(8, 0.25, 2048, 150, seed_extra=slots)
    sched = pk.Schedule(rowpass_slots=slots, single_pass=1)
    say(f"single pass G={slots} split calls")
    a, n1, _ = run(env, inst, sched=sched)
    b, n2, _ = run(env, inst, sched=sched, calls=4)
    c, _, _ = run(env, inst, sched=sched)
    assert n1 == n2 == 150
    assert np.array_equal(a, b) and np.array_equal(a, c)
    acc, nf, s2, _ = oracle.run_instance(inst)
    assert np.all(spectra_err(a, acc) < TOL)


def test_overlap_and_histograms(env):
    """50 % overlap through the single pass over three calls; an integration with level histograms on runs
    the four-step column pass, which counts, for the same instance."""
    torch, pk, dev = env
    N = 1024
    inst = dict(synth.make_correlated_noise(2, 0.3, N, 30, seed_extra=77, window="hann"), hop=N // 2)
    say("single pass with overlap; histograms")
    acc, nf, s2, _ = oracle.run_instance(inst)
    spec, gnf, _ = run(env, inst, calls=3)
    assert gnf == nf == 59
    assert np.all(spectra_err(spec, acc) < TOL)
    plan = pk.Plan([pk.Instance.from_synth(inst)], device=dev)
    packed = torch.from_numpy(inst["packed"]).to(dev)
    half = packed.numel() // 2
    plan.reset()
    plan.set_histograms(True)
    plan.accumulate(packed[:half])
    plan.accumulate(packed[half:])
    spec2, nf2 = plan.spectra()
    counts, _, _ = plan.histograms()
    torch.cuda.synchronize(dev)
    assert nf2 == 59
    assert np.all(spectra_err(spec2.cpu().numpy(), acc) < TOL)
    counted = inst["n_samples"] - N // 2  # the last N - hop samples wait for a next call
    ref = oracle.level_histograms(inst["packed"][:counted * 2 * 2 // 8], 2, 2, counted, inst["pairs"])
    assert np.array_equal(counts.cpu().numpy(), ref)


def test_state_graph_and_grouped_plans(env):
    torch, pk, dev = env
    insts = [synth.make_correlated_noise(8, 0.2, 4096, 50, seed_extra=1),
             synth.make_correlated_noise(2, 0.3, 1 << 16, 6, seed_extra=2),
             synth.make_correlated_noise(4, 0.4, 512, 200, seed_extra=3, window="hann")]
    say("single pass: grouped plan, state export/import, graph replay")
    packed = [torch.from_numpy(d["packed"]).to(dev) for d in insts]
    side = torch.cuda.Stream(dev)
    with torch.cuda.stream(side):
        plan = pk.Plan([pk.Instance.from_synth(d) for d in insts], device=dev, stream=side)
        outs = [torch.zeros((1, 4, d["fft_len"] // 2), dtype=torch.float32, device=dev) for d in insts]
    side.synchronize()

    def integration():
        plan.reset()
        plan.accumulate(packed)
        plan.stokes_all(outs)

    with torch.cuda.stream(side):
        integration()
    side.synchronize()
    eager = [o.clone() for o in outs]
    for i, d in enumerate(insts):
        one = pk.Plan([pk.Instance.from_synth(d)], device=dev)
        one.reset()
        one.accumulate(packed[i])
        assert torch.equal(one.stokes(), eager[i]), i
        # export after the first half, import into a fresh plan, finish there
        h = packed[i].numel() // 2
        one.reset()
        one.accumulate(packed[i][:h])
        state, nf = one.state_export()
        two = pk.Plan([pk.Instance.from_synth(d)], device=dev)
        two.reset()
        two.state_import(state, nf)
        two.accumulate(packed[i][h:])
        assert torch.equal(two.stokes(), eager[i]), i
    plan.graph_capture(integration)
    for r in range(3):
        for o in outs:
            o.zero_()
        torch.cuda.synchronize(dev)
        plan.graph_replay()
        side.synchronize()
        for o, e in zip(outs, eager):
            assert torch.equal(o, e), r


def test_backward_reads_reduced_slots(env):
    """More than 64 slots in use: Stokes and the adjoint read the reduced slot sum (learnable window)."""
    torch, pk, dev = env
    N, F = 1024, 200
    rng = np.random.default_rng(8)
    inst = synth.make_correlated_noise(8, 0.3, N, F, seed_extra=8, window="taps")
    taps = (1 + 0.1 * rng.standard_normal(64)).astype(np.float32)
    g = rng.standard_normal((1, 4, N // 2)).astype(np.float32)
    say("single pass backward with 200 slots in use")
    w, s2 = oracle.window("taps", N, taps=taps.astype(np.float64))
    acc, nf = oracle.accumulate(inst["packed"], 8, 2, inst["n_samples"], N, w, inst["pairs"])
    ref = oracle.stokes(acc, nf, s2)
    gr = oracle.calibrate_backward(inst["packed"], 8, 2, inst["n_samples"], N, w, inst["pairs"], acc, nf, s2,
                                   g.astype(np.float64), taps=taps.astype(np.float64))
    plan = pk.Plan([pk.Instance.from_synth(inst)], device=dev)
    packed = torch.from_numpy(inst["packed"]).to(dev)
    plan.set_window_taps(torch.from_numpy(taps).to(dev))
    plan.reset()
    plan.accumulate(packed)
    st = plan.stokes().cpu().numpy().astype(np.float64)
    grads = plan.calibrate_backward(packed, torch.from_numpy(g).to(dev))
    torch.cuda.synchronize(dev)
    assert np.all(stokes_err(st, ref) < TOL)
    for name, key in (("gain_x", "d_gain_x"), ("gain_y", "d_gain_y")):
        got = grads[name].cpu().numpy().astype(np.float64)
        got = got[..., 0] + 1j * got[..., 1]
        rel = np.max(np.abs(got - gr[key])) / np.max(np.abs(gr[key]))
        assert rel < 1e-5, (name, rel)
    dt = grads["taps"].cpu().numpy().astype(np.float64)
    rel = np.max(np.abs(dt - gr["d_taps"])) / np.max(np.abs(gr["d_taps"]))
    say(f"  taps rel err {rel}")
    assert rel < 1e-4


@pytest.mark.parametrize("log2n", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("bits,streams", [(2, 2), (4, 2), (8, 2), (2, 4), (4, 4), (8, 4)])
def test_word_loads_slots_and_parts(env, log2n, bits, streams):
    """Slots that share a wave and slots without a frame, runs of unequal length, slot counts around the output
    kernel's shares and the chunked reduction; codes read as words (aligned) and item by item (a buffer that starts
    one byte off).  Against the oracle normwise 1e-5; the two loads and split calls bitwise equal."""
    torch, pk, dev = env
    N = 1 << log2n
    rng = synth.rng_for(301, log2n, bits, streams)
    for slots, F in ((1, 3), (2, 5), (8, 3), (64, 67), (128, 66), (128, 200)):
        ts = rng.standard_normal((F * N, streams)) * (16.0 if bits == 8 else 1.0)
        ts[:, -1] += 0.5 * ts[:, 0]
        inst = synth.gen._instance(synth.pack_codes(synth.quantize(ts, bits), bits), bits, streams, N, F, window="hann")
        acc, _, _, _ = oracle.run_instance(inst)
        sched = pk.Schedule(rowpass_slots=slots, single_pass=1)
        say(f"N=2^{log2n} bits={bits} streams={streams} slots={slots} frames={F}")
        spec, nf, st = run(env, inst, sched)
        assert nf == F and np.all(spectra_err(spec, acc) < TOL)
        split, _, _ = run(env, inst, sched, calls=2)
        assert np.array_equal(split, spec)
        plan = pk.Plan([pk.Instance.from_synth(inst)], device=dev, schedules=[sched])
        raw = torch.zeros(inst["packed"].size + 1, dtype=torch.uint8, device=dev)
        raw[1:] = torch.from_numpy(inst["packed"]).to(dev)
        plan.reset()
        plan.accumulate(raw[1:])
        off, _ = plan.spectra()
        assert np.array_equal(off.cpu().numpy(), spec)


@pytest.mark.parametrize("slots", [64, 512])
def test_state_of_fewer_slots_refused(env, slots):
    """A state has its plan's slots: one of half as many is refused before it is read."""
    torch, pk, dev = env
    inst = pk.Instance(fft_len=1 << 10, bits=2)
    plan = pk.Plan([inst], device=dev, schedules=[pk.Schedule(rowpass_slots=slots, single_pass=1)])
    less = pk.Plan([inst], device=dev, schedules=[pk.Schedule(rowpass_slots=slots // 2, single_pass=1)])
    less.accumulate(torch.zeros(2 * (1 << 10) * 4 // 8, dtype=torch.uint8, device=dev))
    state, n = less.state_export()
    with pytest.raises(ValueError):
        plan.state_import(state, n)
    less.state_import(state, n)


@pytest.mark.parametrize("log2n,precision,frames", [(12, "fp32", 700), (12, "fp32", 300), (16, "fp16", 41), (16, "fp16", 3)])
def test_untagged_states_of_fewer_slots_resume(env, log2n, precision, frames):
    """States without a layout in the slots that default plans once had (half as many in a single pass, one with 16-bit
    passes), with every slot in use and with some unused: a resumed integration has the sums of an uninterrupted one
    (FP64 additions in another order, at most frames x 2^-53 of a sum of like signs; the cross products by their
    geometric mean power)."""
    torch, pk, dev = env
    say(f"N=2^{log2n} {precision}, {frames} frames before the export")
    N, more = 1 << log2n, 5
    inst = pk.Instance(fft_len=N, bits=8, precision=precision)
    packed = torch.randint(0, 256, (2 * N * (frames + more),), dtype=torch.uint8, device=dev)
    first, rest = packed[:2 * N * frames], packed[2 * N * frames:]
    whole, plan = pk.Plan([inst], device=dev), pk.Plan([inst], device=dev)
    whole.accumulate(first)
    if precision == "fp32":
        half = pk.Plan([inst], device=dev, schedules=[pk.Schedule(rowpass_slots=256)])
        half.accumulate(first)
        state, n = half.state_export()
        old = state[:-64]
    else:
        state, n = whole.state_export()
        slots = plan._state_parts(0)[1][5]
        assert slots > 1
        sums = state[:-64].view(torch.float64).view(slots, -1)[:min(slots, -(-frames // plan._state_parts(0)[1][6]))]
        old = sums.sum(0).contiguous().view(torch.uint8)
    plan.state_import(old, n)
    whole.accumulate(rest)
    plan.accumulate(rest)
    (want, nw), (got, ng) = whole.spectra(), plan.spectra()
    assert nw == ng == frames + more
    w, g = want[0], got[0]
    scale = torch.stack((w[0], w[1], (w[0] * w[1]).sqrt(), (w[0] * w[1]).sqrt()))
    assert float(((g - w).abs() / scale).max()) < 4 * nw * 2.0 ** -53


def test_states_of_other_layouts_refused(env):
    """More slots than the plan's, and the same size in another split, read back from the device."""
    torch, pk, dev = env
    inst = pk.Instance(fft_len=1 << 13, bits=8)
    data = torch.randint(0, 256, (2 << 14,), dtype=torch.uint8, device=dev)
    make = lambda *s: pk.Plan([inst], device=dev, schedules=[pk.Schedule(*s)])
    wide, few, other = make(7, 0, 0, 0, 8), make(7, 0, 0, 0, 4), make(6, 0, 0, 0, 4)
    states = []
    for p in (wide, few, other):
        p.accumulate(data)
        states.append(p.state_export())
    assert states[1][0].numel() == states[2][0].numel()
    for i, p in enumerate((wide, few, other)):
        for j, (state, n) in enumerate(states):
            say(f"plan {i}, state {j}")
            if i != j:
                with pytest.raises(ValueError):
                    p.state_import(state, n)
        before = p.spectra()[0].clone()
        p.reset()
        p.state_import(*states[i])
        assert torch.equal(p.spectra()[0], before)


@pytest.mark.parametrize("log2n,bound", [(8, 5.2e-8), (9, 5.1e-8), (10, 6.1e-8), (11, 6.5e-8), (12, 6.4e-8)])
def test_rounding_of_constants_does_not_add_up(env, log2n, bound):
    """Integrated power of white noise against 64 bits, rms over channels of the relative error.  Over many frames the
    rounding of the data averages out and that of the transform's constants stays; the bounds are what an FP32 model of
    passes of radix 8 leaves (a 16-point pass with every constant rounded to nearest leaves 6.6e-8 .. 9.7e-8)."""
    torch, pk, dev = env
    F = (1 << 21) >> log2n
    inst = synth.make_correlated_noise(8, 0.3, 1 << log2n, F, seed_extra=900 + log2n)
    acc, _, _, _ = oracle.run_instance(inst)
    plan = pk.Plan([pk.Instance.from_synth(inst)], device=dev)
    plan.accumulate(torch.from_numpy(inst["packed"]).to(dev))
    got = plan.spectra()[0].cpu().numpy()
    rel = (got[0, :2] - acc[0, :2]) / acc[0, :2]
    e = float(np.sqrt(np.mean(rel[:, 1:] ** 2)))
    say(f"N=2^{log2n}, {F} frames: {e:.2e}")
    assert e < bound
