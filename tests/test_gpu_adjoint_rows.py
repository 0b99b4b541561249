"""The adjoint's rank-2 pass on rows that start at any element, at the edges of its
vectors and lane groups, against NumPy in FP64.

With s_max = 0 the call writes dY = X lambda and dX = r lambda^T - (X lambda) beta^T
for lambda = H_hat^{-1} w, which it also returns.  The dots accumulate in FP64
(|error| <= (d + 2) u64 sum |x||v|) and every output is rounded once to its type.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53
U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


@pytest.mark.parametrize("dtype,gdtype", [(np.float32, torch.float32), (np.float32, torch.float64),
                                          (np.float64, torch.float64), (np.float64, torch.float32)])
@pytest.mark.parametrize("d,pad,shift", [(1, 0, 1), (2, 1, 0), (3, 0, 0), (4, 0, 1), (5, 0, 0),
                                         (16, 0, 0), (17, 3, 0), (33, 0, 1), (64, 1, 0), (101, 0, 0),
                                         (255, 0, 0), (256, 3, 1), (511, 0, 0), (512, 0, 0)])
def test_adjoint_of_rows_at_any_element(G, dtype, gdtype, d, pad, shift):
    n = 2531
    g = np.random.default_rng(d)
    flat = torch.from_numpy(g.standard_normal(n * (d + pad) + shift).astype(dtype)).to("cuda:0")
    X = flat[shift:].view(n, d + pad)[:, :d]
    Y = torch.from_numpy(g.standard_normal(n).astype(dtype)).to("cuda:0")
    beta, w = g.standard_normal(d), g.standard_normal(d)
    p = G.Params(kind="srht", seed=2, m=[d + 1], a=[0], r=d + 40, s_max=0,
                 precision="mixed" if dtype == np.float32 else "f64")
    dX, dY, lam = G.backward(X, Y, p, torch.from_numpy(beta).to("cuda:0"),
                             torch.from_numpy(w).to("cuda:0"), grad_dtype=gdtype)
    lam = lam.cpu().numpy()
    Xd, Yd = X.cpu().numpy().astype(np.float64), Y.cpu().numpy().astype(np.float64)
    u, r = Xd @ lam, Yd - Xd @ beta
    eu = (d + 2) * U64 * (np.abs(Xd) @ np.abs(lam))
    er = (d + 3) * U64 * (np.abs(Yd) + np.abs(Xd) @ np.abs(beta))
    ug = U32 if gdtype == torch.float32 else U64
    assert np.all(np.abs(dY.cpu().numpy() - u) <= eu + ug * np.abs(u))
    ref = np.outer(r, lam) - np.outer(u, beta)
    mag = np.outer(np.abs(r), np.abs(lam)) + np.outer(np.abs(u), np.abs(beta))
    tol = np.outer(er, np.abs(lam)) + np.outer(eu, np.abs(beta)) + 4 * (ug + U64) * mag
    assert np.all(np.abs(dX.cpu().numpy() - ref) <= tol)
