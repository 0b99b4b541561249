"""The FP32 / FP64 Gaussian sketch at the edges of its 16-column tiles and column
blocks, of its 64- and 128-row blocks and of its sub-ranges of data rows, on rows
that start at any element, within the bounds of test_gpu_gaussian (every entry
against the oracle on the same operands)."""
import numpy as np
import pytest
import torch

from oracle import rng as R
from test_gpu_gaussian import _case, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


@pytest.mark.parametrize("form", ["f32", "f64"])
@pytest.mark.parametrize("N,d,m,r", [
    (37, 1, [2], 3),             # one step with a ragged end, one column tile
    (513, 15, [64], 65),         # d + 1 = 16; 64 and 128 sketch rows per block
    (1000, 16, [65], 130),       # Y alone in the second tile
    (700, 31, [63], 129),
    (700, 47, [128], 64),
    (9000, 48, [100], 192),      # two splits in sub-ranges, the last one short
    (600, 79, [200], 100),
    (600, 111, [40], 120),
    (600, 143, [150], 160),
    (500, 207, [30], 210),       # 13 tiles: the widest FP64 block
    (500, 208, [30], 220),       # FP64: two column blocks
    (500, 271, [30], 280),       # 17 tiles: the widest FP32 block
    (500, 272, [30], 290),       # both: two column blocks
])
def test_gaussian_tile_edges(G, form, N, d, m, r):
    _case(G, N, d, m, r, form, check_drop=False)


@pytest.mark.parametrize("dtype,u", [(np.float32, 2.0 ** -24), (np.float64, 2.0 ** -53)])
def test_gaussian_of_rows_at_any_element(G, dtype, u):
    # X as the middle of a wider table, one element into its storage; an infinite
    # entry reaches its own column only, rows past the range add nothing
    N, d, m, r = 1003, 33, 96, 70
    g = np.random.default_rng(3)
    T = torch.from_numpy(g.standard_normal(N * (d + 2) + 1).astype(dtype)).to("cuda:0")
    X = T[1:].view(N, d + 2)[:, :d]
    X[N - 1, 7] = float("inf")
    Y = dev(g.standard_normal(N).astype(dtype))
    A, Ah, _ = G.sketch_apply(X, Y, "gaussian", 12, [m], r)
    W = np.concatenate([X.cpu().numpy(), Y.cpu().numpy()[:, None]], 1).astype(np.float64)
    keep = np.arange(d + 1) != 7
    for out, stream, rows in ((A, R.STREAM_G, m), (Ah, R.STREAM_GHAT, r)):
        out = out.cpu().numpy()
        g64 = R.gaussian_block(12, stream, np.arange(rows), np.arange(N))
        ref = g64 @ W[:, keep]
        tol = (N + 16) * u * (np.abs(g64) @ np.abs(W[:, keep]))
        tol += 2.0 ** -16 * (1 + np.abs(g64)) @ np.abs(W[:, keep])
        assert np.all(np.abs(out[:, keep] - ref) <= tol)
        assert np.array_equal(out[:, 7], np.sign(g64[:, N - 1]) * np.inf)


@pytest.mark.parametrize("form", ["f32", "f64"])
@pytest.mark.parametrize("d", [16, 17, 32, 48, 64, 80, 81, 96, 97, 112, 128, 129, 176, 208, 209, 256, 257])
def test_y_beside_the_column_tiles(G, form, d):
    # Y's column is formed beside the tiles of X: widths that fill their tiles, and one more
    _case(G, 530, d, [72], d + 9, form, check_drop=False)


def test_an_infinite_y_stays_in_its_column(G):
    N, d, m, r = 700, 32, 40, 48
    g = np.random.default_rng(4)
    X, Y = dev(g.standard_normal((N, d))), dev(g.standard_normal(N))
    A0, H0, _ = G.sketch_apply(X, Y, "gaussian", 12, [m], r)
    Y[N - 1] = float("inf")
    A, H, _ = G.sketch_apply(X, Y, "gaussian", 12, [m], r)
    for new, old in ((A, A0), (H, H0)):
        assert torch.equal(new[:, :d], old[:, :d])
        assert not torch.isfinite(new[:, d]).any()
