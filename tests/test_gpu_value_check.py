"""The input check inside the evaluation kernels and the filter: one bad value anywhere is
reported, in every kernel family, and -0.0 is not (Sections 2.1, 4.2, 4.5 define the cost
model for finite, non-negative values)."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kr():
    from paper_2601_17654_amd import binding

    return binding


# (kernels, comm kernels, positions, SM choices): the wave kernel's general and fixed
# instances, 64 SM choices (column 1 has no lane of its own), the pair kernel's three, and
# the block kernels behind them (more than 64 SM choices, more than 8 with two comm kernels)
SHAPES = [(5, 1, 6, 3), (32, 1, 33, 32), (9, 1, 4, 64), (24, 1, 25, 16), (7, 2, 6, 5),
          (48, 2, 33, 8), (9, 2, 5, 8), (5, 1, 6, 70), (4, 2, 3, 9)]


def _tables(shape):
    N, M, pos, S = shape
    sp = I.Space(2, N, M, pos, tuple(1 + x % 100 for x in range(S)), (1200.0, 1500.0, 1980.0))
    return sp, I.make_tables(sp, seed=5, comm_bytes=(4e6, 64e6))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N%d-M%d-pos%d-S%d" % s)
def test_every_value_is_checked(kr, shape):
    import torch

    sp, tab = _tables(shape)
    dev = {k: torch.from_numpy(v).cuda() for k, v in tab.items()}
    order = ("t", "pw", "tc", "pc")
    ref = kr.evaluate_and_filter(sp, *(dev[k] for k in order))
    rng = np.random.default_rng(shape[3])
    for k in order:
        n = dev[k].numel()
        cols = shape[3] + 1 if k in ("t", "pw") else shape[3]
        # first, column 1 of the last row, last, and two anywhere
        for x, v in zip((0, n - cols + 1 if cols > 1 else 0, n - 1, *rng.integers(0, n, 2)),
                        (np.nan, np.inf, -1.0, -np.inf, np.nan)):
            bad = dev[k].clone()
            bad.view(-1)[int(x)] = v
            d = [bad if q == k else dev[q] for q in order]
            for call in (kr.evaluate_and_filter, kr.evaluate_partition):
                with pytest.raises(kr.KrError) as e:
                    call(sp, *d)
                assert e.value.status == kr.KR_ENONFINITE, (k, x, v)
    zero = dict(dev, pw=dev["pw"].clone())
    zero["pw"][0, 0, -1, -1] = 0.0
    minus = dict(zero, pw=zero["pw"].clone())
    minus["pw"][0, 0, -1, -1] = -0.0
    a, b = (kr.evaluate_and_filter(sp, *(z[k] for k in order)) for z in (zero, minus))
    assert torch.equal(a.idx, b.idx) and torch.equal(a.T, b.T) and torch.equal(a.E, b.E)
    kr.evaluate_partition(sp, *(minus[k] for k in order))
    again = kr.evaluate_and_filter(sp, *(dev[k] for k in order))
    assert torch.equal(again.idx, ref.idx)


@pytest.mark.parametrize("lens", [(1,), (5000,), (0, 1, 2048, 2049, 0, 7)])
def test_every_point_is_checked(kr, lens):
    import torch

    off = np.concatenate([[0], np.cumsum(lens)])
    rng = np.random.default_rng(3)
    T, E = (torch.from_numpy(rng.uniform(0.1, 1.0, off[-1])).cuda() for _ in range(2))
    kr.pareto_filter(T, E, off)
    for x in {0, int(off[-1]) // 2, int(off[-1]) - 1}:
        for which, v in ((0, np.nan), (1, -1e-300), (0, np.inf)):
            d = [T.clone(), E.clone()]
            d[which][x] = v
            with pytest.raises(kr.KrError) as e:
                kr.pareto_filter(*d, off)
            assert e.value.status == kr.KR_ENONFINITE
        d = [T.clone(), E.clone()]
        d[0][x] = -0.0
        kr.pareto_filter(*d, off)
    assert int(kr.pareto_filter(T[:0], E[:0], [0]).off[0]) == 0  # no segment: still a verdict
