"""The training passes over D (forward step, recomputation, reverse step) at
the edges of their tiles (16-row blocks, 32 columns per wave, 256 per
workgroup, 64-row tiles) and the panel steps between them (64 rows per
workgroup, several times that past 4096 rows), at ranks around the widths of
their products and with padded rows of D, against the FP64 oracle: losses of the forward steps
and every gradient of two unrolled bodies. Tolerances as for the ordinary
sizes: the same FP64 algebra in another order (1e-8); FP32 data and factor
copies (2e-4)."""
import numpy as np
import pytest
import torch

from oracle import accaltproj as A
from oracle import adjoint as J
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu

CASES = [(16, 32, 1), (17, 33, 4), (63, 255, 8), (65, 257, 9), (130, 511, 10), (2064, 30, 3), (4200, 40, 2)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n,r", CASES)
def test_training_passes(m, n, r, dtype):
    print(f"training passes m={m} n={n} r={r} {dtype}", flush=True)
    rng = np.random.default_rng(m + n)
    P, Q = rng.standard_normal((m, r)), rng.standard_normal((n, r))
    T = P @ Q.T
    D = T + np.where(rng.random((m, n)) < 0.1, rng.uniform(-2.0, 2.0, (m, n)) * np.mean(np.abs(T)), 0.0)
    if dtype == torch.float32:
        D = D.astype(np.float32).astype(np.float64)
    U, s, V = A.best_rank_r(T + 0.3 * rng.standard_normal((m, n)), r)
    p = A.Params(r=r, beta=0.5, beta_init=1.0, gamma=0.6, mu=2.0)
    zetas = [0.9 * float(np.max(np.abs(T))) * 0.6 ** k for k in range(2)]
    taus, w = [0.2 * z for z in zetas], [0.5, 1.0]
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    padded = torch.full((m, n + 3), float("nan"), dtype=dtype, device="cuda")   # odd rows, nothing read past n
    padded[:, :n] = dev(D)
    sv = R.Solver(padded[:, :n], r, p.beta, p.beta_init, p.gamma, p.mu, training=True)
    sv.set_state(U, s, V, zetas[0], 0, normD=float(np.linalg.norm(D)))
    losses, ck = sv.unrolled(zetas, taus, w, dev(P), dev(Q))
    got = sv.unrolled_adjoint(ck, zetas, taus, w, dev(P), dev(Q))
    ref = J.unrolled_adjoint(D, U, s, V, zetas, taus, w, p, P, Q)
    tol = 1e-8 if dtype == torch.float64 else 2e-4
    for name, a, b in zip(("losses", "zeta", "U", "sigma", "V"), (losses, *got),
                          (ref.losses, ref.zeta_bar, ref.Ubar0, ref.sbar0, ref.Vbar0)):
        a = a.cpu().numpy() if isinstance(a, torch.Tensor) else np.asarray(a)
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        print(f"  {name} {err:.1e}", flush=True)
        assert err < tol, name
