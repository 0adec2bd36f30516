"""Fused evaluation with more than 256 partitions, where the frontiers are merged in several
launches, against the oracle: a partition whose candidates are one unit still holds several
frontiers when its slab has more than one chunk or tile of candidates, or when the unit spans
several frequencies."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu

# (partitions, frequencies, kernels, comm kernels, positions, SM choices)
SHAPES = [(300, 1, 32, 1, 33, 40),   # one wave per slab, two chunks
          (300, 1, 24, 1, 25, 64),
          (300, 1, 40, 1, 41, 32),   # three chunks
          (300, 1, 10, 2, 11, 9),    # a block per slab, three tiles
          (2048, 3, 5, 1, 6, 70),    # a unit of three frequencies
          (300, 1, 6, 1, 7, 8),      # one chunk: the unit is the partition's frontier
          (300, 2, 6, 2, 7, 3)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "P%d-F%d-N%d-M%d-pos%d-S%d" % s)
def test_many_partitions_match_the_oracle(oracle_lib, shape):
    import torch

    from paper_2601_17654_amd import binding as kr

    P, F, N, M, pos, S = shape
    sp = I.Space(P, N, M, pos, tuple(range(1, S + 1)), tuple(np.linspace(1005.0, 1980.0, F)))
    tab = I.make_tables(sp, seed=N + S, comm_bytes=(4e6, 2e9))
    order = ("t", "pw", "tc", "pc")
    fr = kr.evaluate_and_filter(sp, *(torch.from_numpy(tab[k]).cuda() for k in order))
    off, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    T, E = fr.T.cpu().numpy(), fr.E.cpu().numpy()
    ref = oracle_lib.evaluate_and_filter(sp, *(tab[k] for k in order))
    # the library fixes the order of every fp64 operation: equal to the bit
    assert np.array_equal(off, np.concatenate([[0], np.cumsum([len(r[0]) for r in ref])]))
    for p, (ix, rT, rE) in enumerate(ref):
        s = slice(off[p], off[p + 1])
        assert np.array_equal(idx[s], ix), p
        assert np.array_equal(T[s], rT) and np.array_equal(E[s], rE), p


@pytest.mark.parametrize("n_seg", [1, 260], ids=["one launch", "stages"])
@pytest.mark.parametrize("n", [2_200_000, 4_400_000])
@pytest.mark.parametrize("how", ["few", "some"])
def test_many_units(oracle_lib, n, how, n_seg):
    """A segment of more units than a block has threads, or than its LDS has room for: a point
    or two of each, and a few of each (more than a merge in LDS takes)."""
    import torch

    from paper_2601_17654_amd import binding as kr

    rng = np.random.default_rng(n)
    T = rng.uniform(1.0, 2.0, n)
    E = T + rng.uniform(0.0, 1e-6, n) if how == "few" else rng.uniform(1.0, 2.0, n)
    off = np.concatenate([[0], np.full(n_seg - 1, 5), [n - 5 * (n_seg - 1)]]).cumsum()
    fr = kr.pareto_filter(torch.from_numpy(T).cuda(), torch.from_numpy(E).cuda(), off)
    o, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    for g in range(n_seg):
        s = slice(off[g], off[g + 1])
        assert np.array_equal(idx[o[g]:o[g + 1]], oracle_lib.pareto(T[s], E[s])), g
