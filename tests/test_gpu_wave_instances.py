"""The wave kernel's instances against the oracle: chunks of 4 to 8 positions, general and with
the SM choices fixed, with tables small enough for four waves per SIMD, larger ones, and slabs
of an odd number of doubles."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu

# (kernels, positions, SM choices)
SHAPES = [(24, 16, 16), (24, 20, 16), (24, 24, 16), (28, 28, 16), (32, 32, 16),  # four waves
          (40, 16, 16), (40, 20, 16), (40, 24, 16), (40, 28, 16), (40, 32, 16),
          (25, 16, 16), (27, 28, 16), (31, 32, 16),                              # odd slabs
          (30, 30, 8), (38, 38, 8), (46, 46, 8), (54, 54, 8), (62, 62, 8),
          (80, 54, 8), (90, 62, 8), (24, 8, 32), (24, 10, 32), (24, 12, 32), (24, 14, 32),
          (24, 16, 32), (33, 31, 17)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N%d-pos%d-S%d" % s)
def test_instances_match_the_oracle(oracle_lib, shape):
    import torch

    from paper_2601_17654_amd import binding as kr

    N, pos, S = shape
    sp = I.Space(3, N, 1, pos, tuple(range(1, S + 1)), (1005.0, 1400.0, 1700.0, 1980.0))
    tab = I.make_tables(sp, seed=N + S, comm_bytes=(4e6, 4e9))
    order = ("t", "pw", "tc", "pc")
    fr = kr.evaluate_and_filter(sp, *(torch.from_numpy(tab[k]).cuda() for k in order))
    off, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    T, E = fr.T.cpu().numpy(), fr.E.cpu().numpy()
    for p, (ix, rT, rE) in enumerate(oracle_lib.evaluate_and_filter(sp, *(tab[k] for k in order))):
        s = slice(off[p], off[p + 1])
        # the library fixes the order of every fp64 operation: equal to the bit
        assert np.array_equal(idx[s], ix), p
        assert np.array_equal(T[s], rT) and np.array_equal(E[s], rE), p
