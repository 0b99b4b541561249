"""An infinite coefficient gives infinite gradients, not NaN: rows past a block's share
and columns past a lane's add nothing, not 0 * inf.

X > 0 and beta > 0 with one entry +inf: every residual is -inf, so every entry of
X^T (Y - X beta) is -inf and the residual norm +inf; in the adjoint, dY does not
depend on beta and dX's columns of finite coefficients are r lambda_k = -inf lambda_k.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _data(n, d, dtype, col):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X = torch.rand(n, d, generator=g, device="cuda", dtype=dtype) + 0.1
    Y = torch.randn(n, generator=g, device="cuda", dtype=dtype)
    beta = torch.rand(d, generator=g, device="cuda", dtype=torch.float64) + 0.1
    beta[col] = float("inf")
    return X, Y, beta


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("d", [1, 16, 33, 64, 101, 128, 512, 1000])
@pytest.mark.parametrize("n", [1, 63, 700, 9001])
def test_gradient(G, dtype, d, n):
    for col in (0, d - 1):
        X, Y, beta = _data(n, d, dtype, col)
        for call in (G.fused_resid_grad, G.fused_resid_grad_noalloc):
            g, rn = call(X, Y, beta)
            assert torch.all(g == -float("inf")) and rn.item() == float("inf")


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("d", [2, 5, 16, 33, 64, 100, 101, 130, 330, 512])
def test_adjoint(G, dtype, d):
    n = 2531
    for col in (0, d - 2, d - 1):
        X, Y, beta = _data(n, d, dtype, col)
        w = torch.randn(d, device="cuda", dtype=torch.float64)
        p = G.Params(kind="srht", seed=2, m=[d + 1], a=[0], r=d + 40, s_max=0,
                     precision="mixed" if dtype == torch.float32 else "f64")
        dX, dY, lam = G.backward(X, Y, p, beta, w, grad_dtype=torch.float64)
        ref = X.double().cpu() @ lam.cpu()
        tol = (d + 3) * U64 * (X.double().cpu() @ lam.cpu().abs())
        assert torch.all((dY.cpu() - ref).abs() <= tol)
        keep = torch.arange(d, device="cuda") != col
        want = (-float("inf") * lam.sign()).expand(n, d)
        assert torch.equal(dX[:, keep], want[:, keep])
