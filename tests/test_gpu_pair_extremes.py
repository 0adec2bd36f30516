"""Two comm kernels with powers near the largest finite value: times and energies stay finite,
but the weights that pick what second-phase pairs are compared with do not.  Frontiers equal
the oracle's to the bit all the same."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 9, 3), (12, 13, 4), (5, 6, 8), (68, 66, 1)],
                         ids=lambda s: "N%d-pos%d-S%d" % s)
def test_powers_of_1e308(oracle_lib, shape):
    import torch

    from paper_2601_17654_amd import binding as kr

    N, pos, S = shape
    P, rng = 100, np.random.default_rng(1)
    sp = I.Space(P, N, 2, pos, tuple(range(4, 4 * S + 1, 4)), (1980.0,))
    t0 = rng.uniform(1e-4, 1e-2, (P, 1, N, 1))
    tab = dict(t=t0 * rng.uniform(1, 2, (P, 1, N, S + 1)),
               pw=rng.uniform(2e307, 1e308, (P, 1, N, S + 1)),
               tc=rng.uniform(1e-4, 5e-2, (P, 1, 2, S)), pc=rng.uniform(2e307, 1e308, (P, 1, 2, S)))
    order = ("t", "pw", "tc", "pc")
    fr = kr.evaluate_and_filter(sp, *(torch.from_numpy(tab[k]).cuda() for k in order))
    off, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    T, E = fr.T.cpu().numpy(), fr.E.cpu().numpy()
    for p in range(P):
        rT, rE = oracle_lib.evaluate_partition(sp, *(tab[k] for k in order), p)
        assert np.isfinite(rT).all() and np.isfinite(rE).all()
        ix = oracle_lib.pareto(rT, rE)
        s = slice(off[p], off[p + 1])
        assert np.array_equal(idx[s], ix), p
        assert np.array_equal(T[s], rT[ix]) and np.array_equal(E[s], rE[ix]), p
