"""The streaming passes at the edges of their tiles: last columns that fill no
vector, no lane or no tile, odd row strides (nothing past a row's end is read),
rows that fill no batch or no 16-row tile, against FP64 products of the same
data. Bars: 1e-12 (FP64) and 1e-5 (FP32) of the product's norm; the BF16 form
rounds both operands of the residual part's products (8 significant bits,
relative 2^-8 each), so entry by entry 2^-7 (1 + 2^-9) of the sum of magnitudes,
and FP32's rounding."""
import numpy as np
import pytest
import torch

from paper_1711_05519_amd import rpca as R

pytestmark = pytest.mark.gpu

CASES = [(16, 34, 1, 0), (17, 255, 2, 1), (70, 256, 3, 3), (65, 257, 5, 1), (33, 259, 6, 2), (130, 515, 8, 5),
         (67, 1026, 11, 1), (300, 770, 16, 3)]


@pytest.mark.parametrize("form", ["f64", "f32", "mixed"])
@pytest.mark.parametrize("m,n,r,pad", CASES)
def test_tangent_products_at_tile_edges(m, n, r, pad, form):
    print(f"pass edges m={m} n={n} r={r} pad={pad} {form}", flush=True)
    dtype = torch.float64 if form == "f64" else torch.float32
    rng = np.random.default_rng(m * n)
    cast = lambda X: X.astype(np.float32).astype(np.float64) if form != "f64" else X
    A, B = cast(rng.standard_normal((m, r))), cast(rng.standard_normal((n, r)))
    Ut, Vt = (cast(np.linalg.qr(rng.standard_normal((k, r)))[0]) for k in (m, n))
    D = cast(A @ B.T + rng.standard_normal((m, n)))
    X = D - A @ B.T
    a = np.sort(np.abs(X).ravel())
    gap = np.argmax(np.diff(a[a.size // 4: 3 * a.size // 4])) + a.size // 4   # no entry near the threshold
    zeta = 0.5 * (a[gap] + a[gap + 1])
    S = np.where(np.abs(X) > zeta, X, 0.0)
    dev = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    Db = torch.full((m, n + pad), float("nan"), dtype=dtype, device="cuda")
    Db[:, :n] = dev(D)
    sv = R.Solver(Db[:, :n], r, 1.0, 1.0, 0.5, 1.0, mixed=form == "mixed")
    Y1, Y2, res = sv.tangent_products(dev(A), dev(B), zeta, dev(Ut), dev(Vt))
    E = np.abs(X - S)
    for got, ref, size in ((Y1, (D - S) @ Vt, E @ np.abs(Vt)), (Y2, (D - S).T @ Ut, E.T @ np.abs(Ut))):
        err = np.abs(got.cpu().numpy() - ref)
        if form == "mixed":
            assert np.all(err <= 2.0 ** -7 * (1.0 + 2.0 ** -9) * size + 1e-5 * np.linalg.norm(ref))
        else:
            assert np.linalg.norm(err) <= (1e-12 if form == "f64" else 1e-5) * np.linalg.norm(ref)
    E2 = float(np.sum((X - S) ** 2))
    assert abs(res - E2) <= (1e-12 if form == "f64" else 1e-5) * E2
