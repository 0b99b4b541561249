"""The BF16 Gaussian sketch in every width of its column blocks (64, 128, 192, 256, 320,
448 and 576 columns) and with 64 and 128 sketch rows per block, within the bounds of
test_gpu_gaussian (every compared entry against the oracle on the same rounded operands)."""
import numpy as np
import pytest
import torch

from bounds import bf16_uncertain
from oracle import rng as R
from oracle import sketch as S
from test_gpu_gaussian import U32, _case, _ranges, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


@pytest.mark.parametrize("d", [1, 62, 63, 64, 127, 128, 191, 192, 255, 256, 319, 320, 383, 384, 447,
                               448, 575, 576])
def test_block_widths(G, d):
    # 1003 rows: 15 steps of 64 and a short one; sketch rows that fill no block
    _case(G, 1003, d, [70], d + 9, "bf16", check_drop=False)


@pytest.mark.parametrize("d", [192, 255, 256, 319])
def test_tall_blocks(G, d):
    # 128 sketch rows per block: 64 blocks of them in eight splits (from 512 on); rows
    # at the edges of the 16-row tiles and blocks, the last block short
    N, m, r = 32768 + 37, 8130, d + 9
    splits = G.debug_gaussian_plan(N, d, m, True)
    assert -(-m // 128) * splits >= 512
    rows = np.array([0, 15, 16, 63, 64, 111, 112, 127, 128, 1000, 4095, 8063, 8064, 8127, 8129])
    g = np.random.default_rng(d)
    X = g.standard_normal((N, d)).astype(np.float32)
    Y = g.standard_normal(N).astype(np.float32)
    A, _, _ = G.sketch_apply(dev(X), dev(Y), "gaussian", 88, [m], r, bf16=True)
    out = A[torch.from_numpy(rows).to(A.device)].cpu().numpy()
    assert torch.isfinite(A).all()
    W = S.joint(S.round_to(X, "bf16"), S.round_to(Y, "bf16"))
    g64 = R.gaussian_block(88, R.STREAM_G, rows, np.arange(N))
    gq = S.round_to(g64, "bf16")
    unc, ulp = bf16_uncertain(g64, 2.0 ** -16 * (1.0 + np.abs(g64)))
    ranges = _ranges(N, splits, True)
    n_add = max(b - a for a, b in ranges) * 17 // 16 + len(ranges) + 16
    tol = n_add * U32 * (np.abs(gq) @ np.abs(W)) + np.where(unc, ulp, 0.0) @ np.abs(W)
    assert np.all(np.abs(out[:, : d + 1] - gq @ W) <= tol)
