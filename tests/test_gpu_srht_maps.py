"""The SRHT's index maps against its definition, row by row of a sketch.

Row t of A is the sum over j of H[sigma(t), j] D_j W[pi(j)] with
H[i, j] = (-1)^popcount(i & j), W = [X|Y] padded with zeros, and row t of A_hat
the same with sigma_hat; pi, sigma, sigma_hat and D come from the library's
definition of the streams, evaluated entry by entry.  X and Y hold small whole
numbers, so every sum is exact in FP64 (and in FP32 while it stays below 2^24)
and the rows have to agree in every bit.

Lengths: every padded length of one pass and the smallest of several, odd and
even p, rows per block from 2 to 32768, the last length whose networks
are tabulated and the first whose are not.
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


def _parity(v):
    for s in (16, 8, 4, 2, 1):
        v = v ^ (v >> s)
    return v & 1


def _rows(G, X, Y, seed, p, stream, ts):
    n = 1 << p
    dev = X.device
    pi = G.debug_stream(1, seed, 2, p, 0, n)
    D = G.debug_stream(3, seed, 0, 0, 0, n)
    j = torch.arange(n, device=dev)
    W = torch.cat([X, Y[:, None]], 1).double()
    src = torch.where(pi < X.shape[0], pi, 0)
    Wp = W[src] * ((pi < X.shape[0]).double() * D.double())[:, None]
    out = []
    for t in ts:
        row = int(G.debug_stream(1, seed, stream, p, t, 1)[0])
        out.append(((1 - 2 * _parity(j & row)).double()[:, None] * Wp).sum(0))
    return torch.stack(out)


def _check(G, N, d, p, dtype, seed=11):
    g = torch.Generator(device="cuda").manual_seed(N)
    top = 1 << p
    assert top // 2 < N <= top
    X = torch.randint(-1, 2, (N, d), generator=g, device="cuda").to(dtype)
    Y = torch.randint(-1, 2, (N,), generator=g, device="cuda").to(dtype)
    mK = max(1, N // 2)
    r = min(max(d + 1, N // 3), d + 64)
    A, Ah, _ = G.sketch_apply(X, Y, "srht", seed, [mK], r)
    for out, stream, rows in ((A, 3, mK), (Ah, 4, r)):
        ts = sorted({0, 1, rows // 2, rows - 1} & set(range(rows)))
        ref = _rows(G, X, Y, seed, p, stream, ts)
        assert torch.equal(out[ts, : d + 1].double(), ref), (N, d, stream)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("p", [2, 3, 5, 6, 7, 8, 9, 10, 12, 13, 14, 15, 17])
def test_maps_of_every_length(G, p, dtype):
    _check(G, (1 << p) - (p > 4), 1 if p < 6 else 3, p, dtype)


@pytest.mark.parametrize("p,d,dtype", [(13, 32, torch.float32), (14, 16, torch.float64),
                                       (17, 64, torch.float32)])
def test_maps_with_y_on_its_own(G, p, d, dtype):
    _check(G, (1 << p) - 333, d, p, dtype)


@pytest.mark.slow
@pytest.mark.parametrize("p", [24, 25])
def test_maps_at_the_end_of_the_tables(G, p):
    _check(G, (1 << (p - 1)) + 12345, 1, p, torch.float32)
