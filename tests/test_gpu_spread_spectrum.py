"""The factors of a step stay orthonormal to FP64 when the singular values of the
2r x 2r matrix of Section 2.1 are far apart. Its one-sided SVD ends after a sweep
whose angles are all below 1e-8; a rotation that leaves a part d of its coupling
phi sigma_i^2 then leaves d phi sigma_i / sigma_j between the left vectors i and j.

The states are exact: coordinate bases, and D = [C 0; 0 0] with C upper
triangular, C_ii = sigma_i and C_ij = phi_ij sigma_i, phi below 1e-8, so that the
first sweep is the last and everything before the SVD is free of rounding. What
may remain is the rounding of the rotations and of the two products that form
the factors (r FP64 values of size 1 each), and, from r = 3 on, the couplings that
a sweep's rotations bring back into each other, at most 2 (r - 2) phi^2 sigma_1 / sigma_r."""
import numpy as np
import pytest
import torch

from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


@pytest.mark.parametrize("r,spread", [(2, 1e2), (2, 1e3), (2, 1e4), (3, 1e4), (5, 1e3), (12, 1e2)])
def test_factors_stay_orthonormal(r, spread):
    print(f"spread spectrum r={r} sigma_1/sigma_r={spread:g}", flush=True)
    m, n, phi = 70, 53, 8e-9 if r == 2 else 2e-9
    sig = np.logspace(0.0, -np.log10(spread), r)
    # products of r + 1 terms and the rotations of a sweep, each a few roundings of values of size 1
    bound = 32 * r * EPS + 2 * (r - 2) * phi ** 2 * spread
    for seed in range(8):
        rng = np.random.default_rng(seed)
        C = np.diag(sig)
        for i in range(r):
            C[i, i + 1:] = phi * sig[i] * rng.uniform(0.5, 1.0, r - i - 1) * rng.choice([-1.0, 1.0], r - i - 1)
        D = np.zeros((m, n))
        D[:r, :r] = C
        sv = R.Solver(torch.as_tensor(D, device="cuda"), r, 1.0, 1.0, 0.5, 1.0, trim=False)
        sv.set_state(np.eye(m, r), sig, np.eye(n, r), 1e6, 0, normD=np.linalg.norm(D))
        sv.step()
        U, s, V = (t.cpu().numpy() for t in sv.L_factors())
        assert np.linalg.norm((U * s) @ V.T - D) <= 64 * r * EPS
        for X in (U, V):
            assert np.abs(X.T @ X - np.eye(r)).max() <= bound, seed
