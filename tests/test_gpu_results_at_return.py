"""When a call returns, its results in device memory are there for every stream: a
copy and a kernel on another stream, which waits for nothing, see them."""
import numpy as np
import pytest
import torch

from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["step", "relaxed", "adjoint", "solve", "tangent"])
def test_results_are_there_for_another_stream(call):
    print(f"results at return: {call}", flush=True)
    m, n, r = 3001, 1500, 5
    x = I.gaussian_instance(m, n, r, 0.1, 1.0, seed=9)
    sv = R.Solver(torch.as_tensor(x.D, device="cuda"), r, x.beta, x.beta_init, x.gamma, x.mu_in, training=True)
    P, Q = torch.as_tensor(x.P, device="cuda"), torch.as_tensor(x.Q, device="cuda")
    sv.init()
    start = sv.get_state()
    z = [start[3], 0.7 * start[3]]
    tau = [0.2 * v for v in z]
    ck = sv.unrolled(z, tau, [1.0, 1.0], P, Q)[1]

    def run():
        if call == "adjoint":
            return sv.unrolled_adjoint(ck, z, tau, [1.0, 1.0], P, Q)[1:]
        if call == "tangent":
            U, s, V = start[:3]
            return sv.tangent_products(U * s, V, z[0], U, V)[:2]
        if call == "step":
            sv.step()
        elif call == "relaxed":
            sv.relaxed_step(z[0], tau[0], P, Q)
        else:
            sv.solve()
        return sv.L_factors()

    other = torch.cuda.Stream()
    host = [torch.empty(t.shape, dtype=t.dtype, pin_memory=True) for t in (start[0], start[1], start[2])]
    for rep in range(20):
        sv.put_state(start)
        torch.cuda.synchronize()
        out = run()
        with torch.cuda.stream(other):
            moved = [t + 0.0 for t in out]
            for h, t in zip([host[0], host[1], host[2]] if len(out) == 3 else [host[0], host[2]], out):
                h.copy_(t, non_blocking=True)
        other.synchronize()
        copied = [h.clone() for h in (host if len(out) == 3 else (host[0], host[2]))]
        torch.cuda.synchronize()
        for t, a, b in zip(out, moved, copied):
            assert torch.equal(t, a) and torch.equal(t.cpu(), b) and bool(np.isfinite(b.numpy()).all()), rep
