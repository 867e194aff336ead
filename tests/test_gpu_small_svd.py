"""The SVD of the 2r x 2r matrix of Section 2.1 at every rank (every number of
column pairs, rows per lane and group width of the wave that runs it): one
FP64 step against the oracle, and the same step on a D scaled by a power of
two, whose squares are far from 1 (the SVD works on a scaled copy, so the
results only scale)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


def gpu_step(x, D, st, scale):
    sv = R.Solver(torch.as_tensor(D * scale, device="cuda"), x.r, x.beta, x.beta_init, x.gamma, x.mu_in)
    sv.set_state(st.U, st.sigma * scale, st.V, st.zeta * scale, st.k, normD=O.frobenius(D) * scale)
    sv.step()
    U, s, V = (t.cpu().numpy() for t in sv.L_factors())
    return ((U * (s / scale)) @ V.T, sv.state.zeta / scale, sv.state.sigma1_pt / scale, sv.state.sigma_r1_pt / scale,
            sv.state.err, U, V)


@pytest.mark.parametrize("r", range(1, 17))
def test_step_at_every_rank(r):
    print(f"step r={r}", flush=True)
    x = I.gaussian_instance(90, 74, r, 0.05, 1.0, seed=40 + r)
    p = O.Params(r=r, beta=x.beta, beta_init=x.beta_init, gamma=x.gamma, mu=x.mu_in, tol=1e-8)
    st = O.initialize(x.D, p)
    st.zeta *= 0.5   # the threshold acts, so the complements are not small
    ref = O.step(x.D, st, p)
    L, zeta, s1, sr1, err, U, V = gpu_step(x, x.D, st, 1.0)
    assert np.linalg.norm(L - ref.L()) <= 1e-10 * np.linalg.norm(ref.L())
    assert zeta == pytest.approx(ref.zeta, rel=1e-10)
    assert s1 == pytest.approx(ref.sigma_M[0], rel=1e-11)
    assert sr1 == pytest.approx(ref.sigma_M[r], rel=1e-8)
    assert err == pytest.approx(ref.err, rel=1e-9)
    for X in (U, V):   # the rotations keep the factors orthonormal
        assert np.linalg.norm(X.T @ X - np.eye(r)) <= 1e-12
    for scale in (2.0 ** 300, 2.0 ** -300):
        Ls, zs, s1s, sr1s, errs, _, _ = gpu_step(x, x.D, st, scale)
        assert np.linalg.norm(Ls - L) <= 1e-12 * np.linalg.norm(L)
        assert (zs, s1s, sr1s, errs) == pytest.approx((zeta, s1, sr1, err), rel=1e-12)
