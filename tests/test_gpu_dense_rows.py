"""Dense outputs whose rows are whole memory sectors and ones whose rows are not
(stored and tiled differently): the same bits, whichever of L and S is which."""
import numpy as np
import pytest
import torch

from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("m,n,r", [(2, 16, 1), (37, 128, 6), (130, 272, 7), (1500, 1040, 3), (600, 2064, 10)])
def test_whole_and_ragged_rows_agree(m, n, r, dtype):
    print(f"dense rows m={m} n={n} r={r} {dtype}", flush=True)
    rng = np.random.default_rng(m + n)
    D = torch.as_tensor(rng.standard_normal((m, n)), dtype=dtype, device="cuda")
    sv = R.Solver(D, r, 1.0, 1.0, 0.5, 1.0)
    U, V = rng.standard_normal((m, r)), rng.standard_normal((n, r))
    sv.set_state(U, np.ones(r), V, 1.0, 0)
    L, S = sv.materialize()   # strides of n: whole sectors
    eps = torch.finfo(dtype).eps
    ref, size = U @ V.T, np.abs(U) @ np.abs(V).T   # both factors rounded once, r products and sums
    assert np.all(np.abs(L.double().cpu().numpy() - ref) <= (r + 2) * eps * size)
    x = D - L
    assert torch.equal(S, torch.where(x.abs() > 1.0, x, torch.zeros_like(x)))
    for pads in ((1, 1), (0, 3), (5, 0)):
        A, B = (torch.full((m, n + p), 7.0, dtype=dtype, device="cuda") for p in pads)
        R.rpca_materialize(D, sv.params, sv.state, A[:, :n], B[:, :n], sv.ws)
        assert torch.equal(A[:, :n], L) and torch.equal(B[:, :n], S)
        assert torch.all(A[:, n:] == 7.0) and torch.all(B[:, n:] == 7.0)
        shifted = torch.full((m * n + 1,), 7.0, dtype=dtype, device="cuda")[1:].view(m, n)   # base off a sector
        R.rpca_materialize(D, sv.params, sv.state, shifted, None, sv.ws)
        assert torch.equal(shifted, L)
