"""A call that fails while its report is still on the way keeps its status slot: a later
call does not take that report for its own.

While some stream is captured in global mode the runtime refuses to be asked about
any stream, so a step that waits behind a long kernel returns RPCA_EHIP with its
kernels still queued. The next step, behind a longer kernel on another stream, has to
return its own results."""
import ctypes
import time

import numpy as np
import pytest
import torch

from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


def solver(seed):
    x = I.gaussian_instance(120, 90, 3, 0.1, 1.0, seed=seed)
    sv = R.Solver(torch.as_tensor(x.D, device="cuda"), 3, x.beta, x.beta_init, x.gamma, x.mu_in)
    sv.init()
    return sv


class Captured:
    """A stream of its own that is captured (mode 0: global, 1: this thread) while the block runs."""

    def __init__(self, mode):
        self.lib, self.mode, self.stream = R.library(), mode, ctypes.c_void_p()   # the library's runtime

    def __enter__(self):
        assert self.lib.hipStreamCreateWithFlags(ctypes.byref(self.stream), 1) == 0
        assert self.lib.hipStreamBeginCapture(self.stream, self.mode) == 0
        return self

    def __exit__(self, *exc):
        graph = ctypes.c_void_p()
        self.lib.hipStreamEndCapture(self.stream, ctypes.byref(graph))
        if graph.value:
            self.lib.hipGraphDestroy(graph)
        self.lib.hipStreamDestroy(self.stream)
        self.lib.hipGetLastError()


def scalars(sv):
    s = sv.state
    return s.zeta, s.err, s.sigma1_pt, s.sigma_r1_pt, s.normD, s.k


def test_a_late_report_is_not_anothers():
    print("report on the way", flush=True)
    first, second = solver(5), solver(6)
    starts = [first.get_state(), second.get_state()]
    want = []
    for sv in (first, second):
        sv.step()
        want.append((scalars(sv), sv.U.clone()))
    first.put_state(starts[0])
    second.put_state(starts[1])
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    torch.cuda._sleep(10_000_000)
    e1.record()
    e1.synchronize()
    per_ms = 10_000_000 / e0.elapsed_time(e1)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s1):
        torch.cuda._sleep(int(300 * per_ms))
        with Captured(0), pytest.raises(R.RpcaError) as e:
            first.step()
        assert e.value.status == R.RPCA_EHIP and not s1.query()   # still behind its kernel
    with torch.cuda.stream(s2):
        torch.cuda._sleep(int(600 * per_ms))
        t = time.perf_counter()
        second.step()
        t = time.perf_counter() - t
    torch.cuda.synchronize()
    assert t > 0.4   # it waited for its own report, not for the one before
    assert scalars(second) == want[1][0] and torch.equal(second.U, want[1][1])
    # and the slot serves again once that report has come
    for _ in range(40):
        first.put_state(starts[0])
        first.step()
        assert scalars(first) == want[0][0]


def test_refused_under_capture_and_then_as_before():
    print("refused under capture", flush=True)
    sv = solver(7)
    start = sv.get_state()
    sv.step()
    want = scalars(sv)
    sv.put_state(start)
    torch.cuda.synchronize()
    for _ in range(40):   # more than there are slots
        with Captured(1) as c, pytest.raises(R.RpcaError) as e:
            R.rpca_step(sv.D, sv.params, sv.state, sv.ws, torch.cuda.ExternalStream(c.stream.value))
        assert e.value.status == R.RPCA_EHIP
    sv.put_state(start)
    sv.step()
    assert scalars(sv) == want and np.isfinite(want[1])
