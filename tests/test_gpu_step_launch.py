"""A narrow solve's update is taken by the next step's pass, in one launch; where
the caller asks for per-iterate errors every update is a launch of its own.

Both run the same sums in the same order, so the iterates have to agree in every
bit, at the edges of the widths and of the partial rows that a pass takes, with
and without a tolerance, from a graph or not, and in the adjoint.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _case(G, N, d, dtype, tol=0.0, graph=False):
    g = torch.Generator(device="cuda").manual_seed(N + d)
    X = torch.randn(N, d, generator=g, device="cuda", dtype=dtype)
    Y = X.sum(1) + torch.randn(N, generator=g, device="cuda", dtype=dtype)
    m = [1 << k for k in range((4 * d).bit_length(), N.bit_length() - 1)]
    p = G.Params(kind="countsketch", seed=3, m=m, a=[2] * len(m), r=6 * d, s_max=14, tol=tol, use_graph=graph,
                 precision="mixed" if dtype == torch.float32 else "f64")
    return X, Y, p


@pytest.mark.parametrize("N,d", [(5000, 1), (5001, 2), (5000, 31), (5000, 32), (5000, 33), (6001, 63),
                                 (6000, 64), (6000, 65), (9000, 127), (9000, 128), (9000, 129),
                                 (40000, 128), (300000, 48)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_one_launch_or_two_give_the_same_iterates(G, N, d, dtype):
    X, Y, p = _case(G, N, d, dtype)
    ref = torch.ones(d, dtype=torch.float64, device="cuda")
    b1, _, t1, s1 = G.solve(X, Y, p, record=True)
    b2, _, t2, s2, _ = G.solve(X, Y, p, record=True, beta_ref=ref)
    assert torch.equal(t1, t2) and torch.equal(s1, s2) and torch.equal(b1, b2)
    assert torch.equal(b1, t1[-1]) and torch.isfinite(t1).all()
    p.use_graph = True
    for _ in range(2):
        b3, _, t3, _ = G.solve(X, Y, p, record=True)
        assert torch.equal(t1, t3) and torch.equal(b1, b3)


@pytest.mark.parametrize("N,d", [(5000, 7), (20000, 64), (30000, 128)])
@pytest.mark.parametrize("graph", [False, True])
def test_the_iteration_ends_at_the_same_step(G, N, d, graph):
    X, Y, p = _case(G, N, d, torch.float64, graph=graph)
    ref = torch.ones(d, dtype=torch.float64, device="cuda")
    _, _, traj, sur = G.solve(X, Y, p, record=True)
    first = sum(p.a)
    # between two steps' estimates, well above rounding
    p.tol = float((sur[first + 4] * sur[first + 5]).sqrt())
    b1, i1 = G.solve(X, Y, p)
    b2, i2, _ = G.solve(X, Y, p, beta_ref=ref)
    assert i1["status"] == i2["status"] == "SLSE_OK"
    assert i1["stage2_steps"] == i2["stage2_steps"] < p.s_max
    last = first + i1["stage2_steps"]
    assert torch.equal(b1, b2) and torch.equal(b1, traj[last])


@pytest.mark.parametrize("d", [5, 64, 128])
def test_adjoint_of_narrow_problems(G, d):
    # lambda solves (X^T X) lambda = w: the residual of the iteration's last step is far
    # below the first's
    X, Y, p = _case(G, 8000, d, torch.float64)
    p.s_max = 40
    beta, _ = G.solve(X, Y, p)
    w = torch.randn(d, device="cuda", dtype=torch.float64)
    _, _, lam = G.backward(X, Y, p, beta, w)
    exact = torch.linalg.solve((X.T @ X).cpu(), w.cpu())
    assert (lam.cpu() - exact).norm() <= 1e-9 * exact.norm()
