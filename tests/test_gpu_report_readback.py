"""The report of a solve is read back through a buffer of fixed size, and the
iteration starts from one launch: reports at and past the buffer's size, and
callers' arrays that alias each other.

Both checks are exact: the report holds values that the trajectory's own arrays
hold too, and an aliased start runs the same kernels on the same numbers.
"""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _case(G, s_max, N=1500, d=9):
    g = torch.Generator(device="cuda").manual_seed(s_max)
    X = torch.randn(N, d, generator=g, device="cuda", dtype=torch.float64)
    Y = X.sum(1) + torch.randn(N, generator=g, device="cuda", dtype=torch.float64)
    m = G.paper_schedule(N, d)
    return X, Y, G.Params(kind="srht", seed=5, m=m, a=[2] * len(m), r=6 * d, s_max=s_max)


@pytest.mark.parametrize("steps", [3, 1015, 1016, 1017, 2100])
def test_report_matches_the_recorded_estimates(G, steps):
    X, Y, p = _case(G, 1)
    p.s_max = steps - sum(p.a)
    if p.s_max < 1:
        p.a, p.s_max = [0] * len(p.m), steps
    _, info, _, sur = G.solve(X, Y, p, record=True)
    first = sum(p.a)
    assert info["stage2_steps"] == p.s_max
    assert info["surrogate0"] == float(sur[first])
    assert info["surrogate_final"] == float(sur[steps - 1])


def test_start_from_arrays_that_the_call_writes(G):
    from paper_2509_06856_amd import _lib as L

    X, Y, p = _case(G, 20)
    d = X.shape[1]
    a, b = torch.randn(2, d, device="cuda", dtype=torch.float64).unbind(0)
    first = sum(p.a)
    ref, _ = G.solve(X, Y, p, beta0=a.clone(), beta_prev=b.clone(), start_step=first + 1)
    for alias in ("beta0", "beta_prev"):
        b0, bp = a.clone(), b.clone()
        out = b0 if alias == "beta0" else bp
        prob = G._problem(X, Y)
        q = p.to_c(d, beta0=b0, start_step=first + 1, beta_prev=bp)
        ctx = G.default_context(0)
        L.check(ctx.lib.slse_solve(ctx.h, ctypes.byref(prob), ctypes.byref(q), out.data_ptr(), None,
                                   torch.cuda.current_stream().cuda_stream))
        assert torch.equal(out, ref), alias
