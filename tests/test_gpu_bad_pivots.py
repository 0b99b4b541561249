"""A column of zeros leaves the other columns' solution alone.

Its pivot is zero and counts as 1, so the preconditioner's row and column of it are
those of the identity, its coefficient stays 0 and every other coefficient converges
to the least-squares solution without that column.  A call that fills a report says
that the pivot was bad; one without a report returns the solution.  Columns at the
edges of the factorization's 16-column halves and 32-column steps.
"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import ols as O
from oracle import slse as OS
from slse_inputs import make_problem

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53
CASES = [(1, 0), (12, 7), (16, 15), (33, 32), (40, 16), (64, 0), (150, 95), (300, 299)]


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _problem(d, col, n=6000):
    p = make_problem("plain_small", n=n, d=d, seed=70 + d)
    X = p.X.copy()
    X[:, col] = 0.0
    ref = np.zeros(d)
    keep = np.arange(d) != col
    if keep.any():
        ref[keep] = O.ols_refined(X[:, keep], p.Y)[0]
    return X, p.Y, ref


def _params(G, d, **kw):
    return G.Params(kind="srht", seed=9, m=[2048], a=[2], r=6 * d + 8, s_max=50, **kw)


@pytest.mark.parametrize("d,col", CASES)
@pytest.mark.parametrize("factor,graph", [("chol", False), ("chol", True), ("qr", False)])
def test_solve_without_a_report(G, d, col, factor, graph):
    X, Y, ref = _problem(d, col)
    beta, _ = G.solve(dev(X), dev(Y), _params(G, d, factor=factor, use_graph=graph), report=False)
    b = beta.cpu().numpy()
    assert b[col] == 0.0
    assert np.linalg.norm(b - ref) <= 1e-10 * np.linalg.norm(ref)


def test_solve_batched_without_a_report(G):
    cases = [c for c in CASES if c[0] <= 256]  # the widest batch of rows at any element
    probs = [_problem(d, col) for d, col in cases]
    ps = [_params(G, d) for d, _ in cases]
    betas, _ = G.solve_batched([dev(X) for X, _, _ in probs], [dev(Y) for _, Y, _ in probs], ps,
                               report=False)
    for (d, col), (_, _, ref), beta in zip(cases, probs, betas):
        b = beta.cpu().numpy()
        assert b[col] == 0.0, d
        assert np.linalg.norm(b - ref) <= 1e-10 * np.linalg.norm(ref), d


@pytest.mark.parametrize("d,col", CASES)
def test_factor_reports_it_and_factors_the_rest(G, d, col):
    from paper_2509_06856_amd import _lib as L

    rows = 2 * d + 60
    A = np.random.default_rng(d).standard_normal((rows, d))
    A[:, col] = 0.0
    Ad = dev(A)
    R = torch.empty((d, d), dtype=torch.float64, device="cuda:0")
    M = torch.empty_like(R)
    ctx = G.default_context(0)
    st = ctx.lib.slse_factor(ctx.h, rows, d, ctypes.c_void_p(Ad.data_ptr()), d, L.SLSE_F64, 1.0,
                             L.SLSE_FACTOR_CHOL, ctypes.c_void_p(R.data_ptr()), d,
                             ctypes.c_void_p(M.data_ptr()), d,
                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == L.SLSE_ESINGULAR
    R, M = R.cpu().numpy(), M.cpu().numpy()
    unit = np.eye(d)[col]
    for a in (R[col], R[:, col], M[col], M[:, col]):
        assert np.array_equal(a, unit)
    keep = np.arange(d) != col
    if not keep.any():
        return
    # the bounds of the factorization's other tests: c d u kappa^2, c = 200
    Rref = O.qr_r(A[:, keep])
    tol = 200 * d * U64 * np.linalg.cond(Rref) ** 2
    Rinv = np.linalg.inv(Rref)
    Mref = Rinv @ Rinv.T
    sub = np.ix_(keep, keep)
    assert np.linalg.norm(R[sub] - Rref) <= tol * np.linalg.norm(Rref)
    assert np.linalg.norm(M[sub] - Mref) <= tol * np.linalg.norm(Mref)
