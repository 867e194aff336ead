"""The slab of a batched instance holds a workspace for every call on it: its size for
shapes of one tile to many (no GPU needed), and single calls on the instances of a
solved batch, in their own slabs, with their neighbours untouched."""
import os

import numpy as np
import pytest
import torch

from paper_1711_05519_amd import inputs as I
from paper_1711_05519_amd import rpca as R


@pytest.mark.parametrize("dtype", [R.RPCA_F64, R.RPCA_F32])
@pytest.mark.parametrize("flags", [0, 2, 4])
def test_slab_holds_the_workspace_of_single_calls(dtype, flags):
    if not os.path.exists(R.LIB_PATH):
        pytest.skip("librpca.so not built")
    if flags & 2 and dtype == R.RPCA_F64:
        pytest.skip("mixed products are for float32")
    import ctypes
    lib = R.library()
    for m in (2, 17, 64, 65, 300, 1000, 2047, 5000, 25344):
        for n in (2, 33, 200, 257, 1000, 2000, 10000):
            for r in (1, 3, 5, 10, 16):
                if 2 * r > min(m, n) or (flags & 4 and r > 10):
                    continue
                p = R.Params(m=m, n=n, ldd=n, r=r, dtype=dtype, beta=0.01, beta_init=0.02, gamma=0.5, mu=2.0, tol=1e-6,
                             max_iter=100, init_block=0, init_max_passes=0, flags=flags, seed=1)
                lay = R.BatchLayout()
                assert lib.rpca_batch_layout_of(ctypes.byref(p), ctypes.byref(lay)) == R.RPCA_OK
                assert lay.off_ws % 256 == 0 and lay.slab_bytes % 256 == 0
                assert lay.slab_bytes - lay.off_ws >= R.rpca_workspace_size(p), (m, n, r)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,r,dtype", [(300, 200, 3, torch.float64), (64, 33, 2, torch.float64),
                                         (300, 200, 3, torch.float32), (1000, 700, 6, torch.float32)])
def test_single_calls_in_a_batch_slab(m, n, r, dtype):
    print(f"single calls in a slab m={m} n={n} r={r} {dtype}", flush=True)
    xs = [I.gaussian_instance(m, n, r, 0.05, 1.0, seed=60 + i, tol=1e-5) for i in range(3)]
    p = xs[0]
    D = torch.stack([torch.as_tensor(x.D, dtype=dtype) for x in xs]).cuda()
    bs = R.BatchSolver(D, r, p.beta, p.beta_init, p.gamma, p.mu_in, tol=p.tol, max_iter=6)
    infos = bs.solve()
    i = 1   # a slab with a neighbour on each side
    outside = torch.cat([bs.slabs[0], bs.slabs[2]]).clone()
    ws = bs.slabs[i, bs.layout.off_ws:]
    sv = R.Solver(D[i].contiguous(), r, p.beta, p.beta_init, p.gamma, p.mu_in, tol=p.tol, max_iter=6)
    sv.set_state(bs.U[i], bs.sigma[i], bs.V[i], infos[i].zeta, infos[i].iterations,
                 normD=float(torch.linalg.norm(D[i].double())))
    st = R.State(U=bs.U[i].data_ptr(), V=bs.V[i].data_ptr(), sigma=bs.sigma[i].data_ptr(), zeta=sv.state.zeta,
                 err=sv.state.err, sigma1_pt=0.0, sigma_r1_pt=0.0, normD=sv.state.normD, k=sv.state.k, init_passes=0)
    L, S = torch.empty_like(D[i]), torch.empty_like(D[i])
    R.rpca_materialize(bs.D[i], bs.params, st, L, S, ws)
    Lw, Sw = sv.materialize()
    assert torch.equal(L, Lw) and torch.equal(S, Sw)
    Ut, Vt = torch.empty_like(bs.U[i]), torch.empty_like(bs.V[i])
    R.rpca_trim(bs.params, st, Ut, Vt, ws)
    Uw, Vw = sv.trim()
    assert torch.equal(Ut, Uw) and torch.equal(Vt, Vw)
    R.rpca_step(bs.D[i], bs.params, st, ws)
    sv.step()
    assert (st.zeta, st.err, st.k) == (sv.state.zeta, sv.state.err, sv.state.k) and np.isfinite(st.err)
    assert torch.equal(bs.U[i], sv.U) and torch.equal(bs.V[i], sv.V)
    assert torch.equal(outside, torch.cat([bs.slabs[0], bs.slabs[2]]))
