"""The launch-timing limit of 2,048 points over all cells belongs to the instance alone: one
beyond it is reported, and one at or below it solved, by itself as well as next to small and to
large instances, though a group of four solves from one pool of points."""

import functools

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu

K1, K2, KMAX = [0, 1] * 9, [1, 0] * 9, 2
LIMITS = (64, 2048, 1024)  # points of a cell, points of all cells, candidates of a cell


@functools.lru_cache(maxsize=None)
def _instances():
    """40 random instances and 3 small ones: operations, the oracle's frontiers, and whether they are within
    the limits."""
    import oracle

    rng, kind = np.random.default_rng(1), K1 + K2
    ops, ref = np.zeros((43, len(kind), 4)), []
    for x in range(43):
        for o, k in enumerate(kind):
            if k:
                ops[x, o, :2] = rng.uniform(2e-4, 4e-3), rng.uniform(80, 200)
            else:
                t, p = rng.uniform(1e-4, 2e-3), rng.uniform(300, 700)
                ops[x, o] = t, p, t * rng.uniform(1.05, 1.6), p * rng.uniform(0.6, 0.95)
        if x >= 40:
            ops[x, :, 2:] = ops[x, :, :2]  # overlaps cost nothing: few points
        ref.append(oracle.launch_dp(K1, K2, ops[x], I.P_STATIC_W, KMAX))
    total = np.array([r[3][1] for r in ref])
    fits = np.array([all(a <= b for a, b in zip(r[3], LIMITS)) for r in ref])
    # instances at the limit, between it and what a group's pool holds, and small ones
    assert (total == LIMITS[1]).any() and ((total > 2048) & (total < 2700)).sum() >= 4
    assert (total < 700).sum() >= 3
    return ops, ref, total, fits


@pytest.mark.parametrize("beside", ["alone", "small", "large", "all"])
def test_limit_is_the_instances_own(oracle_lib, beside):
    import torch

    from paper_2601_17654_amd import binding as kr

    ops, ref, total, fits = _instances()
    order = np.argsort(total, kind="stable")
    near = [x for x in range(43) if 1900 < total[x] < 2900]
    if beside == "all":
        calls = [list(range(43))]
    else:
        mates = {"alone": [], "small": list(order[:3]), "large": list(order[-3:])}[beside]
        calls = [[x] + mates for x in near]
    for call in calls:
        got = kr.launch_timing_frontier(K1, K2, torch.from_numpy(ops[call]).cuda(), I.P_STATIC_W,
                                        KMAX, check=False)
        n, T, S = got.n.cpu().numpy(), got.T.cpu().numpy(), got.sched.cpu().numpy()
        assert int(got.status.item()) == (kr.KR_OK if fits[call].all() else kr.KR_ECAPACITY)
        for i, x in enumerate(call):
            rT, _, rS, _ = ref[x]
            assert n[i] == (len(rT) if fits[x] else -1), (x, total[x])
            if fits[x]:
                np.testing.assert_array_equal(T[i, :len(rT)], rT)
                np.testing.assert_array_equal(S[i, :len(rT)], rS)
