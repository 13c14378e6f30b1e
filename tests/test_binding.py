"""Host side of the Python binding, on the CPU: what reaches the library for the tensors a caller may pass.  The
library is replaced by a recorder, so nothing is launched."""
import ctypes as C
import json
import types

import pytest
import torch

import paper_1412_1256_amd as pk
from paper_1412_1256_amd import autograd, autotune


LIBRARY = pk.lib()


class Recorder:
    """Stands for the library: every function records its arguments and succeeds, but for those
    named real, which are the library's own."""

    def __init__(self, real=()):
        self.calls, self.real = [], real

    def __getattr__(self, name):
        if name in self.real:
            return getattr(LIBRARY, name)

        def call(*args):
            self.calls.append((name, args))
            return 0
        return call

    def named(self, name):
        return [a for n, a in self.calls if n == name]


@pytest.fixture
def recorder(monkeypatch):
    r = Recorder()
    monkeypatch.setattr(pk, "lib", lambda: r)
    return r


def cpu_plan(*instances):
    p = pk.Plan.__new__(pk.Plan)
    p.torch, p.instances, p.device = torch, list(instances), torch.device("cpu")
    p.workspace = torch.empty(256, dtype=torch.uint8)
    p._tuned = False
    p._h = None
    return p


@pytest.mark.parametrize("dtype,count,ok", [
    (torch.float32, 64, True), (torch.float64, 64, True), (torch.int32, 64, True), (torch.float32, 128, False),
    (torch.complex64, 64, False), (torch.complex128, 64, False), (torch.complex64, 32, True),
    (torch.complex128, 32, True)])
def test_window_taps_count_floats(recorder, dtype, count, ok):
    """64 taps are 64 floats: a complex tensor stands for its (re, im) pairs, two floats an element, in the 64-bit
    types, which are converted, and in complex64, whose memory is taken as it is."""
    plan = cpu_plan(pk.Instance(fft_len=1 << 10, bits=8, window="taps", n_taps=64))
    taps = torch.arange(count).to(dtype)
    if not ok:
        with pytest.raises(ValueError):
            plan.set_window_taps(taps)
        assert not recorder.named("ps_set_window_taps")
        return
    plan.set_window_taps(taps)
    (_, inst, ptr), = recorder.named("ps_set_window_taps")
    assert inst == 0
    got = list((C.c_float * 64).from_address(ptr.value))
    want = torch.view_as_real(taps).reshape(-1) if taps.is_complex() else taps
    assert got == want.to(torch.float32).tolist()


@pytest.mark.parametrize("n", [1, 2, 3])
def test_differentiable_stokes_calibrates_instance_0(recorder, n):
    """The differentiable Stokes of a plan are instance 0's: its calibration and output go to the library whatever the
    number of instances, and the other instances, which may have no data, are asked for no output."""
    insts = [pk.Instance(fft_len=1 << 10, bits=8), pk.Instance(fft_len=1 << 9, bits=8), pk.Instance(fft_len=256, bits=2)]
    plan = cpu_plan(*insts[:n])
    packed = [torch.zeros(4096, dtype=torch.uint8)] + [None] * (n - 1)
    gx, gy = torch.ones((1, 512), dtype=torch.complex64), torch.ones((1, 512), dtype=torch.complex64)
    dt = torch.zeros((1, 2), dtype=torch.complex64)
    out = autograd.stokes(plan, packed[0] if n == 1 else packed, gx, gy, dt, psi=0.25)
    assert out.shape == (1, 4, 512) and out.dtype == torch.float32
    (_, ptrs, counts, cal, outs), = recorder.named("ps_accumulate_stokes")
    assert list(counts) == [2048] + [0] * (n - 1)
    assert [ptrs[i] for i in range(n)] == [packed[0].data_ptr()] + [None] * (n - 1)
    assert [outs[i] for i in range(n)] == [out.data_ptr()] + [None] * (n - 1)
    assert (cal[0].gain_x, cal[0].gain_y, cal[0].dterms) == (gx.data_ptr(), gy.data_ptr(), dt.data_ptr())
    assert cal[0].psi == 0.25
    for i in range(1, n):
        assert (cal[i].gain_x, cal[i].gain_y, cal[i].dterms, cal[i].psi) == (None, None, None, 0.0)


@pytest.fixture
def state_plan(monkeypatch):
    """Unbound plans of one instance whose imports are recorded; sizes and layouts are the library's own."""
    class Importer(Recorder):  # keeps the bytes that an import hands over (the buffer may live for the call only)
        def ps_state_import(self, h, inst, ptr, frames):
            n = C.c_size_t()
            assert LIBRARY.ps_state_bytes(h, inst, C.byref(n)) == 0
            got = torch.frombuffer(bytearray(C.string_at(ptr.value, n.value)), dtype=torch.uint8)
            self.calls.append(("ps_state_import", (got, frames)))
            return 0

    r = Importer(real=("ps_state_bytes", "ps_state_layout", "ps_last_error"))
    monkeypatch.setattr(pk, "lib", lambda: r)

    def make(sched=None, **kw):
        p = cpu_plan(pk.Instance(**kw))
        p.stream, p.schedules, h, n = None, [sched], C.c_void_p(), C.c_size_t()
        arr, sarr = (pk._Instance * 1)(p.instances[0].to_c()), (pk._Schedule * 1)((sched or pk.Schedule()).to_c())
        assert LIBRARY.ps_plan_scheduled(arr, sarr, 1, C.byref(h), C.byref(n)) == 0, LIBRARY.ps_last_error()
        p._h = h
        return p

    def taken(plan, buf, n=5):
        """What state_import hands to the library: its bytes, or None when it refuses the state."""
        before = len(r.named("ps_state_import"))
        try:
            plan.state_import(buf, n)
        except ValueError:
            assert len(r.named("ps_state_import")) == before
            return None
        (got, frames), = r.named("ps_state_import")[before:]
        assert frames == n
        return got

    return make, taken  # (a plan's __del__ destroys its handle)


def state_of(plan, tagged=True):
    """A state as the plan would export it, every slot filled with its number plus one (waiting samples: 255)."""
    size, layout = plan._state_parts(0)
    slots, waiting = layout[5], layout[7]
    buf = torch.full((size + 64 * tagged,), 255, dtype=torch.uint8)
    buf[:size - waiting] = (torch.arange(slots) + 1).to(torch.uint8).repeat_interleave((size - waiting) // slots)
    if tagged:
        buf[size:] = torch.tensor(layout).view(torch.uint8)
    return buf


S = pk.Schedule
STATE_PLANS = [(S(rowpass_slots=8), dict(fft_len=256)), (S(rowpass_slots=4), dict(fft_len=256)),
               (S(rowpass_slots=16), dict(fft_len=256)), (S(5, rowpass_slots=8, single_pass=2), dict(fft_len=1 << 10)),
               (S(4, rowpass_slots=8, single_pass=2), dict(fft_len=1 << 10)), (S(rowpass_slots=8), dict(fft_len=256, hop=128)),
               (S(rowpass_slots=4), dict(fft_len=256, n_streams=3, pairs=((0, 1), (1, 2))))]


@pytest.mark.parametrize("a", range(len(STATE_PLANS)))
def test_state_is_taken_by_its_own_layout_only(state_plan, a):
    """Slots (fewer and more), split at the same size, waiting samples and pairs: any other layout's state is refused."""
    make, taken = state_plan
    states = [state_of(make(s, **kw)) for s, kw in STATE_PLANS]
    plan = make(STATE_PLANS[a][0], **STATE_PLANS[a][1])
    for b, state in enumerate(states):
        got = taken(plan, state)
        assert (got is not None) == (a == b), (a, b)
        if a == b:
            assert torch.equal(got, state[:-64])
    longer = torch.cat([states[a][:-64], torch.zeros(4096, dtype=torch.uint8)])
    assert taken(plan, longer) is None and taken(plan, states[a][:-72]) is None


def test_states_without_a_layout(state_plan):
    """A buffer of the accumulators alone, as former builds wrote it: taken where its layout is certain."""
    make, taken = state_plan
    for sched, kw in STATE_PLANS:
        plan = make(sched, **kw)
        assert torch.equal(taken(plan, state_of(plan, tagged=False)), state_of(plan)[:-64])
    # single pass by default: half of today's slots, the rest empty; the waiting samples stay at the end
    for hop in (0, 1 << 11):
        plan, half = make(fft_len=1 << 12, hop=hop), make(S(rowpass_slots=256), fft_len=1 << 12, hop=hop)
        size, layout = plan._state_parts(0)
        assert layout[5] == 512
        old = state_of(half, tagged=False)
        got = taken(plan, old)
        sums = old.numel() - layout[7]
        assert torch.equal(got[:sums], old[:sums]) and torch.equal(got[size - layout[7]:], old[sums:])
        assert not got[sums:size - layout[7]].any()
        assert taken(make(S(rowpass_slots=512), fft_len=1 << 12, hop=hop), old) is None  # slots named: not a default


@pytest.mark.parametrize("frames", [1, 4, 5, 9, 1000])
@pytest.mark.parametrize("log2n", [16, 18])
def test_untagged_states_of_16_bit_plans(state_plan, log2n, frames):
    """One slot, or the plan's number of slots in blocks of four frames (of which a short integration used the first):
    the sums of all used slots, in the first."""
    make, taken = state_plan
    plan = make(fft_len=1 << log2n, precision="fp16")
    size, layout = plan._state_parts(0)
    slots, slot = layout[5], size // layout[5]
    assert slots > 1 and layout[6] > 1
    for former in (1, slots):
        sums = torch.rand(former, slot // 8, dtype=torch.float64)
        used = min(former, (frames + 3) // 4)
        sums[used:] = float("nan")  # never written
        old = sums.reshape(-1).view(torch.uint8)
        got = taken(plan, old, frames).view(torch.float64).view(slots, -1)
        assert torch.equal(got[0], sums[:used].sum(0)) and not got[1:].any()
        assert taken(plan, old[:-8], frames) is None


def test_state_without_a_layout_of_long_rows(state_plan):
    """2^21 points had 2048-point rows and have 4096-point rows at the same size: only a named split tells which."""
    make, _ = state_plan
    plan, named = make(fft_len=1 << 21), make(S(log2_n1=10), fft_len=1 << 21)
    (size, layout), (size2, layout2) = plan._state_parts(0), named._state_parts(0)
    assert size == size2 and layout[3:5] == [512, 4096] and layout2[3:5] == [1024, 2048]
    buf = torch.empty(size, dtype=torch.uint8)
    with pytest.raises(ValueError):
        plan.state_import(buf, 5)
    named.state_import(buf, 5)
    assert len(pk.lib().named("ps_state_import")) == 1


def test_tuned_schedules_belong_to_a_build(monkeypatch, tmp_path):
    """A schedule tuned with another build of the library is not taken from the cache: it is timed again."""
    inst, path = pk.Instance(fft_len=1 << 12), str(tmp_path / "tune.json")
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: types.SimpleNamespace(name="x", gcnArchName="gfx"))
    monkeypatch.setattr(autotune, "_input_ring", lambda *a: [None])
    ranked = []

    def timing(instance, sched, *a, **k):
        ranked.append(sched)
        return abs(sched.rowpass_slots - best.rowpass_slots) + abs(sched.single_pass - best.single_pass)

    monkeypatch.setattr(autotune, "time_schedule", timing)
    for best in (pk.Schedule(6, 0, 0, 0, 64, 1), pk.Schedule(6, 0, 0, 0, 512, 1)):
        monkeypatch.setattr(autotune, "build_id", lambda: f"build{best.rowpass_slots}")
        assert autotune.best_schedule(inst, device="cpu", cache=path) == best
        ranked.clear()
        assert autotune.best_schedule(inst, device="cpu", cache=path) == best and not ranked
    assert len(json.load(open(path))) == 2
    monkeypatch.undo()
    a, b = tmp_path / "a.so", tmp_path / "b.so"
    a.write_bytes(b"one"), b.write_bytes(b"two")
    assert autotune.build_id(str(a)) != autotune.build_id(str(b)) and len(autotune.build_id()) == 16


def test_untagged_state_of_a_tuned_plan(state_plan):
    """A tuner may pick another schedule than it did for the plan that saved the state: refused, unless the schedule is
    the caller's own; states with their layout are compared with it."""
    make, taken = state_plan
    sched = S(5, rowpass_slots=8, single_pass=2)
    for tuned in (False, True):
        plan = make(sched, fft_len=1 << 10)
        plan._tuned = tuned
        assert (taken(plan, state_of(plan, tagged=False)) is None) == tuned
        assert taken(plan, state_of(plan)) is not None
        assert taken(plan, state_of(make(S(4, rowpass_slots=8, single_pass=2), fft_len=1 << 10))) is None
