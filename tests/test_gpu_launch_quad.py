"""Four instances per wave of the launch-timing dynamic program against the oracle, bit for
bit: counts that leave the last wave part-filled, cells past 16 and past 64 candidates next
to small ones in the same wave, exact ties, and the longest runs a row of lanes takes."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu


def _ops(rng, kind, n, how):
    ops = np.zeros((n, len(kind), 4))
    for x in range(n):
        for o, k in enumerate(kind):
            if k:
                ops[x, o, :2] = rng.uniform(2e-4, 4e-3), rng.uniform(80, 200)
                continue
            t, p = rng.uniform(1e-4, 2e-3), rng.uniform(300, 700)
            ops[x, o] = t, p, t * rng.uniform(1.05, 1.6), p * rng.uniform(0.6, 0.95)
        if how == "ties" or (how == "mixed" and x % 4 == 1):
            ops[x] = np.round(ops[x] / 1e-3) * 1e-3  # coarse times: many equal sums
        if how == "mixed" and x % 4 == 2:
            ops[x, :, 2] = ops[x, :, 0]  # no slow-down: overlaps dominate, tiny cells
    return ops


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 37])
@pytest.mark.parametrize("how", ["plain", "ties", "mixed"])
@pytest.mark.parametrize("kinds", [([0, 0, 0, 0, 1, 0, 0, 0, 0, 0, 1],) * 2 + (9,),
                                   ([0, 1] * 5, [1, 0, 0] * 3, 4),
                                   ([0] * 14 + [1], [1] + [0] * 14, 14),   # 16 sources a cell
                                   ([0] * 15 + [1], [1] + [0] * 15, 15)],  # one too many
                         ids=["block", "alternating", "run14", "run15"])
def test_four_instances_a_wave(oracle_lib, kinds, how, n):
    import torch

    from paper_2601_17654_amd import binding as kr

    k1, k2, kmax = kinds
    ops = _ops(np.random.default_rng(n + len(k1)), k1 + k2, n, how)
    got = kr.launch_timing_frontier(k1, k2, torch.from_numpy(ops).cuda(), I.P_STATIC_W, kmax,
                                    check=False)
    T, E = got.T.cpu().numpy(), got.E.cpu().numpy()
    S, size = got.sched.cpu().numpy(), got.n.cpu().numpy()
    for x in range(n):
        rT, rE, rS, (cell, total, cand) = oracle_lib.launch_dp(k1, k2, ops[x], I.P_STATIC_W, kmax)
        if cell > 64 or total > 2048 or cand > 1024:
            assert size[x] == -1, x
            continue
        assert size[x] == len(rT), x
        np.testing.assert_array_equal(T[x, :len(rT)], rT)
        np.testing.assert_array_equal(E[x, :len(rT)], rE)
        np.testing.assert_array_equal(S[x, :len(rT)], rS)
