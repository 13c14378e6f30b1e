"""Host side of the Python binding, on the CPU: what reaches the library for the tensors a caller may pass.  The
library is replaced by a recorder, so nothing is launched."""
import ctypes as C

import pytest
import torch

import paper_1412_1256_amd as pk
from paper_1412_1256_amd import autograd


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
