"""The panel steps of the relaxed iterations, the reverse sweep and the cross products
of tangent_products: their last workgroup's sums are the same in every bit from one
repeat to the next, from one workgroup a side to the most a side has (64)."""
import numpy as np
import pytest
import torch

from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


def instance(m, n, r, dtype):
    x = I.gaussian_instance(m, n, r, 0.05, 1.0, seed=70 + r)
    sv = R.Solver(torch.as_tensor(x.D, dtype=dtype, device="cuda"), r, x.beta, x.beta_init, x.gamma, x.mu_in,
                  training=True)
    sv.init()
    return x, sv


@pytest.mark.parametrize("m,n,r,dtype", [
    (40, 33, 2, torch.float64),
    (900, 4097, 5, torch.float64),
    (5000, 300, 10, torch.float32),
])
def test_training_repeats_agree_in_every_bit(m, n, r, dtype):
    print(f"training repeats m={m} n={n} r={r} {dtype}", flush=True)
    x, sv = instance(m, n, r, dtype)
    P, Q = torch.as_tensor(x.P, device="cuda"), torch.as_tensor(x.Q, device="cuda")
    start = sv.get_state()
    z = [start[3], 0.6 * start[3], 0.4 * start[3]]
    tau = [0.2 * v for v in z]
    first = None
    for rep in range(6):
        sv.put_state(start)
        losses, ck = sv.unrolled(z, tau, [1.0] * 3, P, Q)
        zb, Ub, sb, Vb = sv.unrolled_adjoint(ck, z, tau, [1.0] * 3, P, Q)
        got = [torch.tensor(losses), torch.tensor(list(zb)), Ub, sb, Vb] + [t for c in ck for t in c]
        assert all(bool(torch.isfinite(t).all()) for t in got)
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first)), rep


@pytest.mark.parametrize("m,n,r,dtype", [
    (40, 33, 2, torch.float64),
    (3000, 20000, 5, torch.float64),
    (9000, 5000, 11, torch.float32),
])
def test_tangent_products_repeat_in_every_bit(m, n, r, dtype):
    print(f"tangent repeats m={m} n={n} r={r} {dtype}", flush=True)
    rng = np.random.default_rng(r)
    D = torch.as_tensor(rng.standard_normal((m, n)), dtype=dtype, device="cuda")
    sv = R.Solver(D, r, 1.0, 1.0, 0.5, 1.0)
    A, B, U, V = (torch.as_tensor(rng.standard_normal((k, r)), device="cuda") for k in (m, n, m, n))
    first = None
    for rep in range(6):
        Y1, Y2, res = sv.tangent_products(A, B, 1.0, U, V)
        first = first or (Y1, Y2, res)
        assert torch.equal(Y1, first[0]) and torch.equal(Y2, first[1]) and res == first[2], rep
