"""The residual-gradient pass on rows that start at any element, at the edges of
its vectors, lane groups and row steps, against NumPy in FP64; and the update
step on both sides of the width up to which one block takes it.

Bound per column: every product and every addition of a column's sum rounds
once relative to the sum of magnitudes, so
|err| <= 4 (n + d) u |X|^T (|Y| + |X| |beta|).
"""
import numpy as np
import pytest
import torch

from oracle import slse as OS
from slse_inputs import make_problem

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _rows(n, d, pad, shift, dtype, seed):
    """X as the first d columns of a table of d + pad, `shift` elements into its storage."""
    g = np.random.default_rng(seed)
    flat = torch.from_numpy(g.standard_normal(n * (d + pad) + shift).astype(dtype)).to("cuda:0")
    X = flat[shift:].view(n, d + pad)[:, :d]
    Y = torch.from_numpy(g.standard_normal(n).astype(dtype)).to("cuda:0")
    return X, Y, g.standard_normal(d)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("d,pad,shift", [(1, 0, 0), (2, 0, 1), (3, 0, 0), (4, 1, 1), (5, 0, 0),
                                         (31, 0, 1), (32, 1, 0), (33, 3, 1), (101, 0, 0), (128, 0, 1),
                                         (129, 0, 0), (256, 31, 1), (333, 0, 0), (511, 0, 1),
                                         (1023, 0, 0), (1024, 1, 0)])
@pytest.mark.parametrize("n", [1, 63, 700, 9001])
def test_grad_of_rows_at_any_element(G, dtype, d, pad, shift, n):
    X, Y, beta = _rows(n, d, pad, shift, dtype, 1000 * d + n)
    g, rn = G.fused_resid_grad(X, Y, torch.from_numpy(beta).to("cuda:0"), scale=0.5)
    Xd, Yd = X.cpu().numpy().astype(np.float64), Y.cpu().numpy().astype(np.float64)
    r = Yd - Xd @ beta
    mag = np.abs(Yd) + np.abs(Xd) @ np.abs(beta)
    tol = 4 * (n + d) * U64 * 0.5
    assert np.all(np.abs(g.cpu().numpy() - 0.5 * (Xd.T @ r)) <= tol * (np.abs(Xd).T @ mag))
    assert abs(rn.item() - 0.5 * (r @ r)) <= tol * (mag @ mag)


@pytest.mark.parametrize("col", [0, 96, 98, 100])
def test_an_infinite_entry_stays_infinite(G, col):
    # the elements that a moved last chunk reads a second time add nothing, not 0 * inf
    n, d = 5000, 101
    X, Y, beta = _rows(n, d, 0, 0, np.float32, col)
    X = X.abs() + 0.1
    X[4321, col] = float("inf")
    beta = np.abs(beta) + 0.1
    g, rn = G.fused_resid_grad(X, Y, torch.from_numpy(beta).to("cuda:0"))
    assert torch.all(g == -float("inf")) and rn.item() == float("inf")


@pytest.mark.parametrize("d", [47, 48, 49, 128])
def test_update_step_widths(G, d):
    prob = make_problem("plain_small", n=6000, d=d)
    m, r = [1024, 2048], 6 * d
    params = G.Params(kind="srht", seed=5, m=m, a=[2, 2], r=r, s_max=12)
    _, _, traj, sur = G.solve(torch.from_numpy(prob.X).to("cuda:0"),
                              torch.from_numpy(prob.Y).to("cuda:0"), params, record=True)
    _, ref, _ = OS.slse_frs(prob.X, prob.Y, 5, "srht", m, [2, 2], r, s=12)
    tg = traj.cpu().numpy()
    for t in range(len(ref)):
        assert np.linalg.norm(tg[t] - ref[t]) <= 1e-12 * max(np.linalg.norm(ref[t]), 1e-300), t
    assert torch.isfinite(sur).all()
