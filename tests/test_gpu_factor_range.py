"""slse_factor on FP64 data far from 1: entries whose squares leave the range while
those of sqrt(scale) A do not.

R against LAPACK's Householder R of sqrt(scale) A with the bounds of the other factor
tests (c d u kappa^2 for the Cholesky route, c d u kappa for the QR route, c = 200).
"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import ols as O

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _factor(G, A, scale, method, want_M):
    from paper_2509_06856_amd import _lib as L

    rows, d = A.shape
    Ad = torch.from_numpy(A).to("cuda:0")
    R = torch.empty((d, d), dtype=torch.float64, device="cuda:0")
    M = torch.empty_like(R) if want_M else None
    ctx = G.default_context(0)
    L.check(ctx.lib.slse_factor(ctx.h, rows, d, ctypes.c_void_p(Ad.data_ptr()), d, L.SLSE_F64,
                                scale, L.SLSE_FACTOR_QR if method == "qr" else L.SLSE_FACTOR_CHOL,
                                ctypes.c_void_p(R.data_ptr()), d,
                                ctypes.c_void_p(M.data_ptr() if want_M else None), d,
                                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    return R.cpu().numpy(), M.cpu().numpy() if want_M else None


@pytest.mark.parametrize("method", ["chol", "qr"])
@pytest.mark.parametrize("rows,d", [(40, 1), (70, 17), (300, 64), (900, 200)])
@pytest.mark.parametrize("size,scale", [(530, 2.0 ** -1000), (530, 3.0 * 2.0 ** -901),
                                        (-600, 5.0 * 2.0 ** 1001), (-540, 2.0 ** 900), (0, 0.7)])
def test_scale_brings_the_squares_into_range(G, method, rows, d, size, scale):
    A = np.ldexp(np.random.default_rng(rows + d).standard_normal((rows, d)), size)
    R, M = _factor(G, A, scale, method, True)
    Rref = O.qr_r(np.sqrt(scale) * A)
    kappa = np.linalg.cond(Rref)
    tol = 200 * d * U64 * (kappa if method == "qr" else kappa ** 2)
    unit = np.abs(Rref).max()
    assert np.linalg.norm(R / unit - Rref / unit) <= tol * np.linalg.norm(Rref / unit)
    Rinv = np.linalg.inv(Rref / unit)
    Mref = Rinv @ Rinv.T
    Mu = M * unit * unit
    assert np.linalg.norm(Mu - Mref) <= 200 * d * U64 * kappa ** 2 * np.linalg.norm(Mref)
