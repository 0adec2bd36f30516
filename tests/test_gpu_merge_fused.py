"""The one-launch merge (up to 256 segments) and the one-launch filter of few points against
the oracle, on both sides of their limits: segment counts, points in all, points of one
segment (LDS and chunked), empty segments, ties and duplicates, and a short output."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(rng, n, how):
    if how == "curve":  # nearly every point on the frontier
        T = np.sort(rng.uniform(1.0, 2.0, n))
        E = np.sort(rng.uniform(1.0, 2.0, n))[::-1].copy()
        p = rng.permutation(n)
        return T[p], E[p]
    if how == "ties":
        return rng.integers(1, 30, n) * 0.25, rng.integers(0, 30, n) * 0.25
    return rng.uniform(1.0, 2.0, n), rng.uniform(1.0, 2.0, n)


CASES = [[1], [0, 5, 0], [4096], [4097], [512, 513, 3071], [16] * 256, [16] * 255 + [17],
         [16] * 257, [1] * 256, [2048, 2047, 1, 1], [9000, 30, 0, 5000], [40000] + [7] * 255,
         [3000] * 4, [0] * 256, [2049] * 300]


@pytest.mark.parametrize("lens", CASES, ids=lambda n: "%d-%d" % (len(n), sum(n)))
@pytest.mark.parametrize("how", ["random", "curve", "ties"])
def test_merge_paths(oracle_lib, lens, how):
    import torch

    from paper_2601_17654_amd import binding as kr

    rng = np.random.default_rng(len(lens) + sum(lens))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    T, E = _points(rng, off[-1], how)
    d = [torch.from_numpy(x).cuda() for x in (T, E)]
    fr = kr.pareto_filter(*d, off)
    o, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    gT, gE = fr.T.cpu().numpy(), fr.E.cpu().numpy()
    for g in range(len(lens)):
        s = slice(off[g], off[g + 1])
        ix = oracle_lib.pareto(T[s], E[s]) if lens[g] else np.zeros(0, np.int64)
        w = slice(o[g], o[g + 1])
        assert np.array_equal(idx[w], ix), g
        assert np.array_equal(gT[w], T[s][ix]) and np.array_equal(gE[w], E[s][ix])
    total = int(o[-1])
    if total > 1:  # a short output holds the first points, and the offsets stay whole
        cut = kr.pareto_filter(*d, off, cap=total // 2, sync=False)
        assert np.array_equal(cut.off.cpu().numpy(), o)
        assert np.array_equal(cut.idx.cpu().numpy(), idx[:total // 2])
        assert np.array_equal(cut.T.cpu().numpy(), gT[:total // 2])
