"""The M-IHS update against the oracle's iterates on both sides of each of its rules:
32 / 33 and 64 / 65 columns (the sizes of the one-block update), 128 / 129 (one block or
blocks over M), and 65 to 128 columns with more partial rows than one block sums."""
import numpy as np
import pytest
import torch

from oracle import slse as OS
from slse_inputs import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse

    return slse


def _compare(G, n, d):
    prob = make_problem("plain_small", n=n, d=d)
    m, r = [1024, 2048], 6 * d
    params = G.Params(kind="srht", seed=5, m=m, a=[2, 2], r=r, s_max=12)
    _, _, traj, sur = G.solve(torch.from_numpy(prob.X).to("cuda:0"),
                              torch.from_numpy(prob.Y).to("cuda:0"), params, record=True)
    _, ref, _ = OS.slse_frs(prob.X, prob.Y, 5, "srht", m, [2, 2], r, s=12)
    tg = traj.cpu().numpy()
    for t in range(len(ref)):
        assert np.linalg.norm(tg[t] - ref[t]) <= 1e-12 * max(np.linalg.norm(ref[t]), 1e-300), t
    assert torch.isfinite(sur).all()


@pytest.mark.parametrize("d", [31, 32, 33, 64, 65, 128, 129])
def test_widths(G, d):
    _compare(G, 6000, d)


@pytest.mark.parametrize("d,blocks", [(65, 257), (100, 400), (128, 512), (64, 513)])
def test_rows_summed_ahead_of_the_update(G, monkeypatch, d, blocks):
    # more partial rows than one block sums: 256 from 65 columns on, 512 below
    monkeypatch.setenv("SLSE_RG_BLOCKS", str(blocks))
    _compare(G, 60000, d)
