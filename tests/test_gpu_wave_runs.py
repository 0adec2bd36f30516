"""The wave kernel's split of launch positions into runs and rounds, against the oracle:
every compiled chunk size, runs that start inside an 8-row block, idle lanes, several
chunks per run."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu

# (kernels, positions, SM choices): 64 // S runs per SM choice
SHAPES = [(6, 7, 8), (6, 1, 8), (41, 42, 19), (24, 25, 16), (20, 21, 10), (31, 32, 7), (15, 16, 3),
          (33, 34, 2), (17, 18, 1), (40, 41, 33), (13, 9, 21), (25, 26, 30), (9, 10, 20),
          (28, 29, 24), (30, 12, 32), (11, 12, 32), (47, 48, 64), (8, 9, 31), (16, 17, 12),
          (5, 6, 60), (37, 33, 13)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N%d-pos%d-S%d" % s)
@pytest.mark.parametrize("comm", [(4e6, 64e6), (4e8, 6e9)], ids=["short", "long"])
def test_runs_match_the_oracle(oracle_lib, shape, comm):
    import torch

    from paper_2601_17654_amd import binding as kr

    N, pos, S = shape
    sp = I.Space(3, N, 1, pos, tuple(range(1, S + 1)), (1005.0, 1400.0, 1700.0, 1980.0))
    tab = I.make_tables(sp, seed=N + S, comm_bytes=comm)
    order = ("t", "pw", "tc", "pc")
    fr = kr.evaluate_and_filter(sp, *(torch.from_numpy(tab[k]).cuda() for k in order))
    off, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    T, E = fr.T.cpu().numpy(), fr.E.cpu().numpy()
    for p in range(sp.n_parts):
        rT, rE = oracle_lib.evaluate_partition(sp, *(tab[k] for k in order), p)
        ix = oracle_lib.pareto(rT, rE)
        s = slice(off[p], off[p + 1])
        # the library fixes the order of every fp64 operation: equal to the bit
        assert np.array_equal(idx[s], ix)
        assert np.array_equal(T[s], rT[ix]) and np.array_equal(E[s], rE[ix])
