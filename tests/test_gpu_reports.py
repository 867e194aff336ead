"""Results that a call's last kernel reports through a status slot: from more host
threads than there are slots (32; the calls that find none copy their results), each
on its own stream, equal to the same calls made one after another."""
import threading

import numpy as np
import pytest
import torch

import oracle as O
from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("training", [False, True])
def test_reports_from_many_threads(training):
    print(f"reports training={training}", flush=True)
    x = I.gaussian_instance(120, 90, 3, 0.1, 1.0, seed=5)
    p = O.Params(r=3, beta=x.beta, beta_init=x.beta_init, gamma=x.gamma, mu=x.mu_in, tol=1e-8)
    st = O.initialize(x.D, p)
    D = torch.as_tensor(x.D, device="cuda")
    P, Q = torch.as_tensor(x.P, device="cuda"), torch.as_tensor(x.Q, device="cuda")

    def one(scale):
        sv = R.Solver(D, 3, x.beta, x.beta_init, x.gamma, x.mu_in, training=training)
        sv.set_state(st.U, st.sigma, st.V, scale * st.zeta, st.k, normD=np.linalg.norm(x.D))
        if training:
            res = sv.relaxed_step(scale * st.zeta, 0.2 * st.zeta, P, Q)
            return res.loss, res.dloss_dzeta, res.err, res.sigma1, res.sigma_r1
        sv.step()
        return sv.state.zeta, sv.state.err, sv.state.sigma1_pt, sv.state.sigma_r1_pt, sv.state.k

    scales = [1.0 - 0.01 * i for i in range(40)]
    want = [one(s) for s in scales]
    got = [None] * len(scales)
    start = threading.Barrier(len(scales))
    torch.cuda.synchronize()

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            start.wait(timeout=60)
            for _ in range(3):
                got[i] = one(scales[i])

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(scales))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert got == want
