"""The threshold network's forward and gradient at batch sizes around the
chunks its gradient is summed in, against the FP64 reference formulas."""
import numpy as np
import pytest
import torch

from oracle import learned as Lr
from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 33, 64])
def test_network_batches(B):
    print(f"network B={B}", flush=True)
    rng = np.random.default_rng(B)
    th = (0.4 * rng.standard_normal(R.RPCA_MLP_PARAMS)).astype(np.float32)
    phi = rng.standard_normal((B, 4)).astype(np.float32)
    go = rng.standard_normal(B).astype(np.float32)
    dev = lambda x: torch.as_tensor(x, device="cuda")
    o = R.rpca_mlp_forward(dev(th), dev(phi)).cpu().numpy()
    g = R.rpca_mlp_backward(dev(th), dev(phi), dev(go)).cpu().numpy()
    t64 = th.astype(np.float64)
    acts = [Lr.mlp_forward(t64, phi[b].astype(np.float64)) for b in range(B)]
    ref = sum((Lr.mlp_backward(t64, a[1], float(go[b])) for b, a in enumerate(acts)), np.zeros(R.RPCA_MLP_PARAMS))
    size = sum((np.abs(Lr.mlp_backward(t64, a[1], float(go[b]))) for b, a in enumerate(acts)),
               np.zeros(R.RPCA_MLP_PARAMS))
    # FP32: chains of at most 4 + 32 + B terms, bounded against the largest parameter's sum of magnitudes
    eps = np.finfo(np.float32).eps
    assert np.all(np.abs(o - np.array([a[0] for a in acts])) <= 80 * eps * (1.0 + np.abs(o)) * np.abs(th).sum() / 32)
    assert np.all(np.abs(g - ref) <= (80 + B) * eps * (size + size.max(initial=0.0)))
