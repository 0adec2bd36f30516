"""Launch-timing instances with values that are not numbers, infinite or overflowing: their own
results are unspecified, but calls end, schedules are read back inside the table, and the
instances beside them in a group keep the oracle's results to the bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KINDS = [([0, 0, 1, 0, 1], [0, 1, 0, 0, 1], 3), ([0, 1] * 5, [1, 0, 0] * 3, 4),
         ([0] * 15 + [1], [1] + [0] * 15, 15)]  # runs of 15: the one-instance solver


@pytest.mark.parametrize("p_static", [60.0, 0.0])
@pytest.mark.parametrize("kinds", KINDS, ids=["short", "alternating", "run15"])
def test_bad_values_stay_with_their_instance(oracle_lib, kinds, p_static):
    import torch

    from paper_2601_17654_amd import binding as kr

    k1, k2, kmax = kinds
    rng = np.random.default_rng(5)
    n, nops = 48, len(k1) + len(k2)
    ops = rng.uniform(1e-4, 2e-3, (n, nops, 4))
    ops[:, :, 1::2] = rng.uniform(100, 700, (n, nops, 2))
    bad = np.arange(n) % 3 == 1
    for x, how in zip(np.flatnonzero(bad), np.resize([0, 1, 2, 3, 4], bad.sum())):
        some = rng.random(nops) < 0.5
        if how == 0:
            ops[x, some, 0] = np.nan
        elif how == 1:
            ops[x, some, 2] = np.inf
        elif how == 2:
            ops[x] = np.nan
        elif how == 3:
            ops[x, :, ::2] = 1e308  # finite: the sums overflow, and 0 W times that is no number
        else:
            ops[x, some] = -ops[x, some]
    got = kr.launch_timing_frontier(k1, k2, torch.from_numpy(ops).cuda(), p_static, kmax,
                                    check=False)
    T, S, size = got.T.cpu().numpy(), got.sched.cpu().numpy(), got.n.cpu().numpy()
    assert ((size >= -1) & (size <= 64)).all()
    for x in np.flatnonzero(~bad):
        rT, _, rS, (cell, total, cand) = oracle_lib.launch_dp(k1, k2, ops[x], p_static, kmax)
        assert cell <= 64 and total <= 2048 and cand <= 1024
        assert size[x] == len(rT), x
        np.testing.assert_array_equal(T[x, :len(rT)], rT)
        np.testing.assert_array_equal(S[x, :len(rT)], rS)
