"""The report's phase times: every stage-1 step is counted in ms_stage1.

A solve that ends with stage 1 has an empty stage 2, whose time is the distance of two
events with nothing between them (5.0 us), at every width: up to 128 columns, where a
step's update may be left to the next pass, as beyond, where it never is.  Medians over
many calls; an update of 128 columns between the two events adds 3.9 us, and half of that
is the allowance.
"""
import statistics

import pytest
import torch

pytestmark = pytest.mark.gpu


def _empty_stage2_ms(G, d, calls=60):
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(6000, d, generator=g, device="cuda", dtype=torch.float64)
    Y = torch.randn(6000, generator=g, device="cuda", dtype=torch.float64)
    p = G.Params(kind="countsketch", seed=3, m=[1024], a=[2], r=6 * d, s_max=0)
    ms = [G.solve(X, Y, p)[1]["ms_stage2"] for _ in range(calls)]
    return statistics.median(ms[10:])


def test_no_stage1_step_is_counted_in_stage2():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_06856_amd import slse as G

    empty = _empty_stage2_ms(G, 160)
    assert _empty_stage2_ms(G, 128) <= empty + 2e-3
