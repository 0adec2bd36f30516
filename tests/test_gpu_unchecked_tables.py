"""Unchecked tables with powers that are not numbers: the partition's own frontier is
unspecified, but it takes no more room than it has candidates (one per frequency here), so the
partitions beside it keep the oracle's results to the bit."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pos,S", [(1, 1), (2, 1), (3, 2), (5, 8)])
@pytest.mark.parametrize("P", [3, 300])
@pytest.mark.parametrize("M", [1, 2])
def test_neighbours_are_untouched(oracle_lib, M, P, pos, S):
    import torch

    from paper_2601_17654_amd import binding as kr

    sp = I.Space(P, 4, M, pos, tuple(range(1, S + 1)), tuple(np.linspace(1005.0, 1980.0, 64)))
    tab = I.make_tables(sp, seed=3, comm_bytes=(4e6, 64e6))
    order = ("t", "pw", "tc", "pc")
    ref = oracle_lib.evaluate_and_filter(sp, *(tab[k] for k in order))
    tab["pw"][1::2] = np.nan
    fr = kr.evaluate_and_filter(sp, *(torch.from_numpy(tab[k]).cuda() for k in order),
                                validate=False)
    off, idx, T = fr.off.cpu().numpy(), fr.idx.cpu().numpy(), fr.T.cpu().numpy()
    for p in range(P):
        n = off[p + 1] - off[p]
        assert 0 <= n <= sp.n_cand
        if p % 2 == 0:
            s = slice(off[p], off[p + 1])
            assert np.array_equal(idx[s], ref[p][0]) and np.array_equal(T[s], ref[p][1]), p
