"""The QR route on more rows than 65536 tiles of 32 hold, the most blocks that a grid
takes in its second dimension.

Every entry of the last pass's Gram matrix sums `rows` products, so R is within rows u
kappa of LAPACK's; 32 rows left out would change it by 32 / rows, far more.
"""
import numpy as np
import pytest
import torch

from oracle import ols as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_more_than_2_21_rows(dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse as G

    rows, d = (1 << 21) + 70, 3
    A = np.random.default_rng(21).standard_normal((rows, d)).astype(dtype)
    R, M = G.factor(torch.from_numpy(A).to("cuda:0"), d, 0.5, "qr")
    Rref = O.qr_r(np.sqrt(0.5) * A.astype(np.float64))
    kappa = np.linalg.cond(Rref)
    tol = rows * 2.0 ** -53 * kappa
    assert np.linalg.norm(R.cpu().numpy() - Rref) <= tol * np.linalg.norm(Rref)
    Mref = np.linalg.inv(Rref.T @ Rref)
    assert np.linalg.norm(M.cpu().numpy() - Mref) <= 2 * tol * kappa * np.linalg.norm(Mref)
