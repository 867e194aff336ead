"""A relaxed step on data or from a state with a NaN reports NaN in every singular
value (a finite one would be left over from another launch)."""
import numpy as np
import pytest
import torch

from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 3, 8, 10])
@pytest.mark.parametrize("where", ["D", "state"])
def test_relaxed_step_reports_nan(r, where):
    print(f"non-finite relaxed step r={r} {where}", flush=True)
    x = I.gaussian_instance(140, 110, r, 0.1, 1.0, seed=5)
    P, Q = torch.as_tensor(x.P, device="cuda"), torch.as_tensor(x.Q, device="cuda")
    U, s, Vt = np.linalg.svd(x.P @ x.Q.T)
    U, s, V = U[:, :r].copy(), s[:r].copy(), Vt[:r].T.copy()
    zeta = 0.5 * np.abs(x.D).max()
    good = R.Solver(torch.as_tensor(x.D, device="cuda"), r, 1.0, 1.0, 0.5, x.mu_in, training=True)
    good.set_state(U, s, V, zeta, 0, normD=np.linalg.norm(x.D))
    for _ in range(2):   # a finite step leaves finite values where the next one works
        good.relaxed_step(zeta, 0.2 * zeta, P, Q)
    D = x.D.copy()
    if where == "D":
        D[17, 5] = np.nan
    else:
        U[17, r - 1] = np.nan
    bad = R.Solver(torch.as_tensor(D, device="cuda"), r, 1.0, 1.0, 0.5, x.mu_in, training=True)
    bad.set_state(U, s, V, zeta, 0, normD=np.linalg.norm(x.D))
    res = bad.relaxed_step(zeta, 0.2 * zeta, P, Q)
    assert np.isnan(res.sigma1) and np.isnan(res.sigma_r1) and np.isnan(res.loss)
    assert bool(torch.isnan(bad.sigma).all()), bad.sigma
