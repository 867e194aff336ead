"""The sums that the last workgroup of a launch takes over every workgroup's
partials: a partial that had not reached it (it ran on another XCD, with its own
L2) would differ between repeats. Their order is fixed, so repeats agree in every
bit, from one workgroup a side to more than the device holds at once."""
import pytest
import torch

from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,r,dtype,count", [
    (64, 33, 2, torch.float64, 1),
    (3000, 2999, 5, torch.float64, 1),
    (700, 500, 6, torch.float32, 40),
    (700, 500, 3, torch.float64, 40),
])
def test_repeats_agree_in_every_bit(m, n, r, dtype, count):
    print(f"election m={m} n={n} r={r} {dtype} x{count}", flush=True)
    xs = [I.gaussian_instance(m, n, r, 0.05, 1.0, seed=300 + i, tol=1e-5) for i in range(min(count, 4))]
    p = xs[0]
    D = torch.stack([torch.as_tensor(xs[i % len(xs)].D, dtype=dtype) for i in range(count)]).cuda()
    bs = R.BatchSolver(D, p.r, p.beta, p.beta_init, p.gamma, p.mu_in, tol=p.tol, seed=7)
    first = None
    for rep in range(6):
        got = [(i.iterations, i.err_hist, i.zeta_hist) for i in bs.solve()]
        U, V = bs.U.clone(), bs.V.clone()
        for i in range(len(xs), count):   # the same instance elsewhere in the launch
            assert got[i] == got[i % len(xs)] and torch.equal(U[i], U[i % len(xs)]), (rep, i)
        if first is None:
            first = got, U, V
        assert got == first[0] and torch.equal(U, first[1]) and torch.equal(V, first[2]), rep
