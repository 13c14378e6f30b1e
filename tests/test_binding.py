"""Host side of the Python binding, on the CPU: what reaches the library for the tensors a caller may pass.  The
library is replaced by a recorder, so nothing is launched."""
import ctypes as C

import pytest
import torch

import paper_1412_1256_amd as pk


class Recorder:
    """Stands for the library: every function records its arguments and succeeds."""

    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
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
