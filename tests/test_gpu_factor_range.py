"""slse_factor on FP64 data far from 1: entries whose squares leave the range while
those of sqrt(scale) A do not, and Gram matrices below the normal range.

R against LAPACK's Householder R of sqrt(scale) A with the bounds of the other factor
tests (c d u kappa^2 for the Cholesky route, c d u kappa for the QR route, c = 200).  A
Gram entry below the normal range is rounded by up to 2^-1075 per row of A, which takes
the place of u in the Cholesky route's bound there.  M is asked for where it is in range.
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


@pytest.mark.parametrize("method", ["chol", "qr"])
@pytest.mark.parametrize("d", [1, 16, 20, 33, 64])
@pytest.mark.parametrize("every", [1, 2, 7])
def test_pivots_below_the_normal_range(G, method, d, every):
    # every such column 2^-515 times standard normals, the others of size 1
    rows = 2 * d + 30
    small = np.arange(d) % every == 0
    A = np.random.default_rng(d + every).standard_normal((rows, d))
    A[:, small] *= 2.0 ** -515
    R, _ = _factor(G, A, 1.0, method, False)
    if every == 1:
        Rref = O.qr_r(np.ldexp(A, 515))
        kappa = np.linalg.cond(Rref)
        R = np.ldexp(R, 515)
        # 2^-1075 per row against the Gram's diagonal of rows 2^-1030
        u = U64 if method == "qr" else 2.0 ** -45
        tol = 200 * d * u * (kappa if method == "qr" else kappa ** 2)
        assert np.linalg.norm(R - Rref) <= tol * np.linalg.norm(Rref)
    elif method == "chol":
        # a column of size 2^-515 among others: R's rows scale with the columns
        S = np.where(small, 2.0 ** 515, 1.0)
        Rref = O.qr_r(A * S)
        tol = 200 * d * 2.0 ** -45 * np.linalg.cond(Rref) ** 2
        assert np.linalg.norm(R * S - Rref) <= tol * np.linalg.norm(Rref)
