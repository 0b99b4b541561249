"""The CountSketch's per-wave counts where the last block has fewer waves than the others
and where one, two or four waves' counts fit in a block, on both list routes.

Whole numbers small enough that every sum is exact in either type, so the sketches have to
equal the oracle's.
"""
import numpy as np
import pytest
import torch

from oracle import sketch as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


@pytest.mark.parametrize("sort", ["0", "1"])
@pytest.mark.parametrize("r", [7, 2048, 4096, 4097, 6144, 8192, 8193])
@pytest.mark.parametrize("N", [8200, 16320, 16321, 16385, 16449, 70000])  # 129, 255, 256, 257, 258, 547 waves
def test_counts(G, monkeypatch, sort, r, N):
    monkeypatch.setenv("SLSE_CS_SORT", sort)
    g = np.random.default_rng(N + r)
    X = g.integers(-8, 9, (N, 3)).astype(np.float32)
    Y = g.integers(-8, 9, N).astype(np.float32)
    m = [1024, 2048]
    A, Ah, _ = G.sketch_apply(torch.from_numpy(X).to("cuda:0"), torch.from_numpy(Y).to("cuda:0"),
                              "countsketch", 31, m, r)
    ref = S.countsketch(X.astype(np.float64), Y.astype(np.float64), 31, m, r)
    assert np.array_equal(A.cpu().numpy(), ref["A"])
    assert np.array_equal(Ah.cpu().numpy(), ref["Ahat"])
