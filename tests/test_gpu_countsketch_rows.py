"""The CountSketch's gathers at the edges of their lane groups, vectors and column
passes, on rows that start at any element, against the oracle.

Bound per entry: every addition into a bucket rounds once, so
|err| <= (rows of the largest bucket + 16) u sum |x| over the bucket (16: the parts,
the lane groups and the folds).
"""
import numpy as np
import pytest
import torch

from oracle import rng as R
from oracle import sketch as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _sketch_abs(W, h, rows, m):
    out, n = np.zeros((rows, W.shape[1])), np.bincount(h, minlength=1).max()
    np.add.at(out, h, np.abs(W))
    return out, n


@pytest.mark.parametrize("dtype,u", [(np.float32, 2.0 ** -24), (np.float64, 2.0 ** -53)])
@pytest.mark.parametrize("N,d,pad,shift,m,r", [
    (700, 1, 0, 1, [64, 128, 256], 3),
    (700, 3, 2, 0, [64], 9),
    (5000, 15, 0, 0, [128, 256, 512, 1024, 2048], 96),
    (5000, 16, 1, 1, [512, 1024], 17),
    (3000, 33, 0, 0, [256, 512, 1024], 40),
    (3000, 64, 3, 1, [1024], 384),
    (4000, 127, 0, 0, [512, 1024, 2048], 130),
    (2000, 128, 1, 0, [512, 1024], 200),
    (2000, 129, 0, 1, [512, 1024], 200),   # FP64: two chunks of a row per pass
    (2000, 256, 0, 0, [1024], 300),
    (2000, 257, 0, 0, [512, 1024], 300),   # FP32: the same
    (1500, 513, 0, 1, [1024], 600),
    (1500, 700, 1, 0, [1024], 800),        # several passes
    (40000, 9, 0, 0, [16384], 2),          # two Hessian buckets of 20000 rows
])
def test_countsketch_rows(G, dtype, u, N, d, pad, shift, m, r):
    if r <= d:
        r = d + 1
    g = np.random.default_rng(N + d)
    T = torch.from_numpy(g.standard_normal(N * (d + pad) + shift).astype(dtype)).to("cuda:0")
    X = T[shift:].view(N, d + pad)[:, :d]
    Y = torch.from_numpy(g.standard_normal(N).astype(dtype)).to("cuda:0")
    A, Ah, lay = G.sketch_apply(X, Y, "countsketch", 31, m, r)
    Xd, Yd = X.cpu().numpy().astype(np.float64), Y.cpu().numpy().astype(np.float64)
    ref = S.countsketch(Xd, Yd, 31, m, r)
    W = S.joint(Xd, Yd)
    h, _ = R.countsketch_hash(31, N, m[-1])
    hh, _ = R.countsketch_hash_hat(31, N, r)
    A, Ah = A.cpu().numpy(), Ah.cpu().numpy()
    for i, mi in enumerate(m):
        mag, n = _sketch_abs(W, h & (mi - 1), mi, mi)
        sl = slice(lay["offset"][i], lay["offset"][i] + mi)
        assert np.all(np.abs(A[sl] - ref["A"][sl]) <= (n + 16) * u * mag), mi
    mag, n = _sketch_abs(W, hh, r, r)
    assert np.all(np.abs(Ah - ref["Ahat"]) <= (n + 16) * u * mag)


def test_an_infinite_row_stays_in_its_buckets(G):
    N, d, m, r = 6000, 37, [256, 512, 1024], 50
    g = np.random.default_rng(8)
    X = torch.from_numpy(g.standard_normal((N, d))).to("cuda:0")
    Y = torch.from_numpy(g.standard_normal(N)).to("cuda:0")
    rows = [0, 1234, N - 1]
    X[rows] = float("inf")
    A, Ah, lay = G.sketch_apply(X, Y, "countsketch", 4, m, r)
    h, _ = R.countsketch_hash(4, N, m[-1])
    hh, _ = R.countsketch_hash_hat(4, N, r)
    bad = np.zeros(len(A), bool)
    for i, mi in enumerate(m):
        bad[lay["offset"][i] + (h[rows] & (mi - 1))] = True
    badh = np.zeros(r, bool)
    badh[hh[rows]] = True
    assert np.array_equal(~np.isfinite(A[:, :d].cpu().numpy()).any(1), bad)
    assert np.array_equal(~np.isfinite(Ah[:, :d].cpu().numpy()).any(1), badh)
