"""Status slots: the calls that can do without one (they copy their results then)
do not take those that solves need. 40 relaxed steps are held in flight at once, each
on a stream that waits for one long kernel."""
import threading
import time

import numpy as np
import pytest
import torch

import oracle as O
from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu

HELD = 40   # more than a pool has


class Case:
    def __init__(self):
        x = I.gaussian_instance(120, 90, 3, 0.1, 1.0, seed=5)
        p = O.Params(r=3, beta=x.beta, beta_init=x.beta_init, gamma=x.gamma, mu=x.mu_in, tol=1e-8)
        self.x, self.st = x, O.initialize(x.D, p)
        self.D = torch.as_tensor(x.D, device="cuda")
        self.P, self.Q = torch.as_tensor(x.P, device="cuda"), torch.as_tensor(x.Q, device="cuda")

    def solver(self, training):
        x, st = self.x, self.st
        sv = R.Solver(self.D, 3, x.beta, x.beta_init, x.gamma, x.mu_in, tol=1e-8, training=training)
        sv.set_state(st.U, st.sigma, st.V, st.zeta, st.k, normD=np.linalg.norm(x.D))
        return sv

    def relaxed(self, sv):
        r = sv.relaxed_step(self.st.zeta, 0.2 * self.st.zeta, self.P, self.Q)
        return r.loss, r.dloss_dzeta, r.err, r.sigma1, r.sigma_r1

    def step(self, sv):
        sv.step()
        s = sv.state
        return s.zeta, s.err, s.sigma1_pt, s.sigma_r1_pt, s.k

    def tangent(self, sv):
        U, s, V = sv.L_factors()
        Y1, Y2, res = sv.tangent_products(U * s, V, self.st.zeta, U, V)
        return Y1.cpu().tolist(), Y2.cpu().tolist(), res

    def adjoint(self, sv, ck):
        z = [self.st.zeta] * 2
        zb, Ub, sb, Vb = sv.unrolled_adjoint(ck, z, [0.2 * v for v in z], [1.0, 1.0], self.P, self.Q)
        return list(zb), Ub.cpu().tolist(), sb.cpu().tolist(), Vb.cpu().tolist()


class Held:
    """HELD relaxed steps in flight until a kernel of about `seconds` on another stream ends."""

    def __init__(self, case, seconds=0.8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        torch.cuda._sleep(10_000_000)
        e1.record()
        e1.synchronize()
        self.cycles = int(10_000_000 * seconds * 1e3 / e0.elapsed_time(e1))
        self.case = case
        self.solvers = [case.solver(True) for _ in range(HELD)]
        self.streams = [torch.cuda.Stream() for _ in range(HELD)]
        self.got = [None] * HELD
        torch.cuda.synchronize()

    def __enter__(self):
        gate = torch.cuda.Stream()
        self.open = torch.cuda.Event()
        with torch.cuda.stream(gate):
            torch.cuda._sleep(self.cycles)
            self.open.record()
        ready = threading.Barrier(HELD + 1)

        def work(i):
            with torch.cuda.stream(self.streams[i]):
                self.streams[i].wait_event(self.open)
                ready.wait(timeout=60)
                self.got[i] = self.case.relaxed(self.solvers[i])

        self.threads = [threading.Thread(target=work, args=(i,)) for i in range(HELD)]
        for t in self.threads:
            t.start()
        ready.wait(timeout=60)
        time.sleep(0.1)
        assert not self.open.query()   # the steps are in flight
        return self

    def __exit__(self, *exc):
        for t in self.threads:
            t.join(timeout=60)
        assert not any(t.is_alive() for t in self.threads)


def test_solves_beside_other_calls():
    print("slots: a solve beside held relaxed steps", flush=True)
    c = Case()
    want_relaxed = c.relaxed(c.solver(True))
    want = c.solver(False).solve()
    one, many = c.solver(False), [c.solver(False) for _ in range(3)]
    held = Held(c)
    with held:
        got = one.solve()
        got_many = R.solve_many(many, n_streams=3)
    for g in [got, *got_many]:
        assert (g.status, g.iterations, g.err_hist, g.zeta_hist) == (want.status, want.iterations, want.err_hist,
                                                                     want.zeta_hist)
    assert held.got == [want_relaxed] * HELD


def test_calls_without_a_slot_copy():
    print("slots: calls that find none", flush=True)
    c = Case()
    ck = c.solver(True).unrolled([c.st.zeta] * 2, [0.2 * c.st.zeta] * 2, [1.0, 1.0], c.P, c.Q)[1]
    calls = {"relaxed": lambda sv: c.relaxed(sv), "step": lambda sv: c.step(sv), "tangent": lambda sv: c.tangent(sv),
             "adjoint": lambda sv: c.adjoint(sv, ck)}
    want = {k: f(c.solver(True)) for k, f in calls.items()}
    solvers = {k: c.solver(True) for k in calls}
    streams = {k: torch.cuda.Stream() for k in calls}
    got = {}
    held = Held(c)

    def work(k):
        with torch.cuda.stream(streams[k]):
            got[k] = calls[k](solvers[k])

    with held:
        threads = [threading.Thread(target=work, args=(k,)) for k in calls]
        for t in threads:
            t.start()
        for t in threads:
            t.join(timeout=60)
    assert got == want
