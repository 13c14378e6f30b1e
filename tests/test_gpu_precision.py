"""Precision form on the GPU (16-bit passes on the matrix cores) against the FP64 oracle, through the C ABI.

Error measure per Stokes product P (after Eq. 2, no fitted correction): max_k |P_gpu - P_ref| / I_ref,k.

Tolerances.  Each value is rounded to the 16-bit format three times on its way through the transform (after
the first column stage, into the inter-pass buffer, after the first row stage), with unit roundoff
u = 2^-11 (FP16) or 2^-8 (BF16); the DFT matrices carry hi + lo parts, so their own error is of order u^2.
Per frame a channel's power then has a relative error of a few u, with random sign from frame to frame, so
an integration of F frames averages it down by about 1/sqrt(F); the maximum over 2^17 channels is about 4.5
times the rms.  This gives about 3e-4 (FP16) and 2.5e-3 (BF16) at F = 32.  Bounds: FP16 1e-3 for F >= 32
(the precision form's stated tolerance); BF16 8x that (the ratio of the two roundoffs), 8e-3 for F >= 32.
Unpacking and the FP64 integration are unchanged from the plain path.
"""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

TOL = {"fp16": 1e-3, "bf16": 8e-3}


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_1412_1256_amd as pk
    pk.lib()
    return torch, pk, torch.device("cuda:0")


def run_gpu(env, inst, precision, accum, chunk=0, calls=1):
    torch, pk, dev = env
    plan = pk.Plan([pk.Instance.from_synth(inst, precision=precision, accum=accum, chunk_frames=chunk)], device=dev)
    packed = torch.from_numpy(inst["packed"]).to(dev)
    plan.reset()
    if calls == 1:
        plan.accumulate(packed)
    else:
        per = inst["n_frames"] // calls * inst["fft_len"] * inst["n_streams"] * inst["bits"] // 8
        for c in range(calls):
            end = packed.numel() if c == calls - 1 else (c + 1) * per
            plan.accumulate(packed[c * per:end])
    st = plan.stokes()
    torch.cuda.synchronize(dev)
    return st.cpu().numpy().astype(np.float64)


def ref_stokes(inst):
    acc, nf, s2, _ = oracle.run_instance(inst)
    return oracle.stokes(acc, nf, s2)


def stokes_err(got, ref):
    I = ref[:, 0:1, :]
    return np.max(np.abs(got - ref) / I, axis=2)


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
@pytest.mark.parametrize("accum", ["fp64", "kahan32"])
@pytest.mark.parametrize("log2n", [16, 17, 18])
def test_two_stream_int8(env, precision, accum, log2n):
    say(f"precision {precision} {accum} int8 S=2 N=2^{log2n} F=32")
    inst = synth.make_correlated_noise(8, 0.3, 1 << log2n, 32, seed_extra=log2n)
    ref = ref_stokes(inst)
    got = run_gpu(env, inst, precision, accum)
    e = stokes_err(got, ref)
    say(f"  err I,Q,U,V {e.tolist()}")
    assert np.all(e < TOL[precision])


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_four_streams_two_pairs(env, precision):
    say(f"precision {precision} S=4 pairs (0,2),(1,3) N=2^18 F=48")
    inst = synth.make_precision(n_frames=48)
    ref = ref_stokes(inst)
    got = run_gpu(env, inst, precision, "kahan32")
    e = stokes_err(got, ref)
    say(f"  err per pair, I,Q,U,V {e.tolist()}")
    assert np.all(e < TOL[precision])


@pytest.mark.parametrize("pairs", [((0, 1), (2, 3)), ((3, 1),)])
def test_four_streams_other_pairs(env, pairs):
    """Four int8 streams paired otherwise than (0, 2), (1, 3): each workgroup transforms one pair, taking its
    two streams out of the four-stream word (the (0, 2), (1, 3) layout is transformed two pairs at a time)."""
    say(f"precision fp16 S=4 pairs {pairs} N=2^17 F=96")
    inst = dict(synth.make_precision(n_frames=48), pairs=[list(p) for p in pairs])
    inst = dict(inst, fft_len=1 << 17, n_frames=96)  # the same samples as 2^17-point frames
    ref = ref_stokes(inst)
    got = run_gpu(env, inst, "fp16", "kahan32")
    e = stokes_err(got, ref)
    say(f"  err per pair, I,Q,U,V {e.tolist()}")
    assert np.all(e < TOL["fp16"])


@pytest.mark.parametrize("bits", [2, 4, 32])
def test_other_formats_and_hann(env, bits):
    say(f"precision fp16 bits={bits} Hann N=2^16 F=40")
    inst = synth.make_correlated_noise(bits, 0.2, 1 << 16, 40, seed_extra=bits, window="hann")
    ref = ref_stokes(inst)
    got = run_gpu(env, inst, "fp16", "kahan32")
    e = stokes_err(got, ref)
    say(f"  err I,Q,U,V {e.tolist()}")
    assert np.all(e < TOL["fp16"])


def test_tone_dynamic_range(env):
    """A tone 40 dB above the noise per channel.  The 16-bit rounding of the column pass output scales with
    the tone in the tone's row of the inter-pass buffer, so the channels of that row carry errors relative to
    the tone rather than to their own noise: judged as spurious-free range, max_k |P_gpu - P_ref| over the
    tone's power over every other channel (bound 1e-5, i.e. spurs at least 50 dB below the tone), plus the
    tone channel itself (relative bound of the precision form)."""
    say("precision fp16 tone +40 dB S=4 N=2^18 F=32")
    inst = synth.make_precision(n_frames=32, tone_db=40.0)
    ref = ref_stokes(inst)
    got = run_gpu(env, inst, "fp16", "kahan32")
    k = 43690
    peak = ref[:, 0, k][:, None]
    assert np.all(ref[:, 0, k] > 1e3 * np.median(ref[:, 0, :], axis=1))
    d = np.abs(got - ref)
    d[:, :, k - 1:k + 2] = 0.0  # the tone's own channels are judged below
    sf = np.max(d, axis=2) / peak
    say(f"  max spur / tone per pair {sf.tolist()}")
    assert np.all(sf < 1e-5)
    et = np.abs(got[:, :, k] - ref[:, :, k]) / peak
    say(f"  tone channel err {et.tolist()}")
    assert np.all(et < TOL["fp16"])


def test_chunks_and_calls(env):
    """Frames split into chunks and over calls: same result within the rounding of the FP64 sums."""
    say("precision fp16 chunked 8 frames, 3 calls")
    inst = synth.make_correlated_noise(8, 0.3, 1 << 17, 36, seed_extra=5)
    a = run_gpu(env, inst, "fp16", "kahan32")
    b = run_gpu(env, inst, "fp16", "kahan32", chunk=8, calls=3)
    c = run_gpu(env, inst, "fp16", "kahan32")
    assert np.array_equal(a, c)  # deterministic
    rel = np.max(np.abs(a - b) / a[:, 0:1, :])
    say(f"  chunked vs whole {rel}")
    assert rel < 1e-6


@pytest.fixture(scope="module")
def config3():
    """The precision case at its stated length: 4 int8 streams (2 bands x 2 pols), 2^18 points, 610 frames
    (10 s), and its FP64 oracle Stokes."""
    inst = synth.make_precision(n_frames=610)
    return inst, ref_stokes(inst)


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_precision_config_610_frames(env, config3, precision):
    """Both 16-bit formats with Kahan-compensated integration over the 610 frames: every Stokes product of
    both pairs within 1e-3 of the oracle (per channel, relative to I).  By the estimate above the errors at
    F = 610 are about 6.9e-5 (FP16) and 5.7e-4 (BF16), the 32-frame figures times sqrt(32 / 610)."""
    inst, ref = config3
    say(f"precision case, 610 frames, {precision} + kahan32")
    got = run_gpu(env, inst, precision, "kahan32")
    e = np.max(np.abs(got - ref) / ref[:, 0:1, :], axis=2)
    say(f"  per-Stokes errors {e.tolist()}")
    assert np.all(e < 1e-3), e


@pytest.mark.parametrize("log2n,streams,F,cuts", [(16, 2, 5, (0, 1, 5)), (16, 2, 37, (0, 3, 20, 37)), (17, 4, 19, (0, 6, 19)),
                                                  (16, 4, 300, (0, 300)), (18, 2, 6, (0, 2, 6)), (18, 4, 3, (0, 3))])
@pytest.mark.parametrize("window", ["rect", "hann"])
def test_slots_and_windowed_words(env, log2n, streams, F, cuts, window):
    """The 16-bit row pass's slots (blocks of four frames, fewer blocks than slots, launches that begin inside a block)
    and the windowed word loads, each against item-by-item decoding and against one call: int8 streams in an order
    that the word loader does not take (the pairs swapped) give the same rounding points.  Sums of products of at most
    3e5 terms in FP64 or compensated FP32 and another order of the slots: 1e-6 of the mean power."""
    torch, pk, dev = env
    N = 1 << log2n
    gen = torch.Generator(device=dev).manual_seed(log2n * 100 + F)
    x = (torch.randn((F * N, streams), device=dev, generator=gen) * 16).round().clamp(-128, 127)
    x[:, -1] = (0.5 * x[:, 0] + 0.5 * x[:, -1]).round()
    packed = x.to(torch.int8).view(torch.uint8).reshape(-1)
    pairs = ((0, 1),) if streams == 2 else ((0, 2), (1, 3))
    # one stream more, never used: neither two nor four streams, so the codes are decoded item by item
    wide = torch.cat([x, x[:, :1]], 1).to(torch.int8).view(torch.uint8).reshape(-1).contiguous()

    def spectra(n_streams, data, steps):
        plan = pk.Plan([pk.Instance(fft_len=N, bits=8, n_streams=n_streams, pairs=pairs, window=window, precision="fp16",
                                    accum="kahan32")], device=dev)
        plan.reset()
        for lo, hi in zip(steps, steps[1:]):
            plan.accumulate(data[lo * N * n_streams:hi * N * n_streams])
        return plan.spectra()

    say(f"N=2^{log2n} streams={streams} F={F} {window}")
    got, nf = spectra(streams, packed, cuts)
    one, _ = spectra(streams, packed, (0, F))
    items, _ = spectra(streams + 1, wide, (0, F))
    scale = got[:, :2].mean(dim=2).amax()
    assert nf == F
    assert float((got - one).abs().max() / scale) < 1e-6 and float((items - one).abs().max() / scale) < 1e-6


@pytest.mark.parametrize("log2n,streams,F,cuts", [(16, 2, 3, ()), (16, 2, 16, (5,)), (16, 2, 17, (16,)), (16, 2, 33, (15, 32)),
                                                  (16, 2, 83, (1, 18, 64)), (17, 4, 37, (20, 21)), (18, 2, 50, (31,))])
def test_slot_blocks_sum_every_frame_once(env, log2n, streams, F, cuts):
    """The 16-bit row pass's slots in blocks of sixteen frames: integrations shorter and longer than a block and than all
    slots' blocks, calls that begin and end inside one.  Against the frames integrated one by one, whose spectra are
    added in FP64: the same products, so the sums differ by their order only (F x 2^-53 of the terms' sizes)."""
    torch, pk, dev = env
    N = 1 << log2n
    pairs = ((0, 1),) if streams == 2 else ((0, 2), (1, 3))
    plan = pk.Plan([pk.Instance(fft_len=N, bits=8, n_streams=streams, pairs=pairs, precision="fp16")], device=dev)
    gen = torch.Generator(device=dev).manual_seed(F)
    data = (torch.randn((F, N * streams), device=dev, generator=gen) * 16).clamp(-127, 127).to(torch.int8).view(torch.uint8)
    say(f"N=2^{log2n} streams={streams} F={F} cuts={cuts}")
    want = torch.zeros((len(pairs), 4, N // 2), dtype=torch.float64, device=dev)
    for f in range(F):
        plan.reset()
        plan.accumulate(data[f])
        want += plan.spectra()[0]
    steps = (0,) + cuts + (F,)
    plan.reset()
    for lo, hi in zip(steps, steps[1:]):
        plan.accumulate(data[lo:hi].reshape(-1))
    got, n = plan.spectra()
    cross = (want[:, 0] * want[:, 1]).sqrt()[:, None]
    size = torch.cat((want[:, :2], cross, cross), 1)
    assert n == F and float(((got - want).abs() / size).max()) < 4 * F * 2.0 ** -53
