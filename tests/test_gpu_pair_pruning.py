"""Two comm kernels: dropping the second-phase pairs that cannot be on a frontier leaves every
frontier as the oracle has it, to the bit: position counts around a wave's 64, every number
of SM choices of the kernel, comm kernels from negligible to longer than compute, equal
kernels and SM choices (exact ties between pairs), zero power, and the largest slabs."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu


def _check(oracle, sp, tab):
    import torch

    from paper_2601_17654_amd import binding as kr

    order = ("t", "pw", "tc", "pc")
    fr = kr.evaluate_and_filter(sp, *(torch.from_numpy(tab[k]).cuda() for k in order))
    off, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    T, E = fr.T.cpu().numpy(), fr.E.cpu().numpy()
    for p in range(sp.n_parts):
        rT, rE = oracle.evaluate_partition(sp, *(tab[k] for k in order), p)
        ix = oracle.pareto(rT, rE)
        s = slice(off[p], off[p + 1])
        assert np.array_equal(idx[s], ix), p
        assert np.array_equal(T[s], rT[ix]) and np.array_equal(E[s], rE[ix]), p


@pytest.mark.parametrize("shape", [(48, 33, 8), (20, 21, 8), (9, 1, 8), (11, 12, 7), (6, 7, 1),
                                   (30, 31, 2), (66, 64, 3), (66, 65, 3), (70, 67, 5), (3, 4, 6),
                                   (425, 426, 1)], ids=lambda s: "N%d-pos%d-S%d" % s)
@pytest.mark.parametrize("comm", [(1e3, 1e4), (8e6, 5e8), (4e8, 8e9)],
                         ids=["tiny", "usual", "long"])
def test_pruned_frontiers(oracle_lib, shape, comm):
    N, pos, S = shape
    sp = I.Space(2, N, 2, pos, tuple(range(4, 4 + S)), (1005.0, 1500.0, 1980.0))
    _check(oracle_lib, sp, I.make_tables(sp, seed=N + S, comm_bytes=comm))


@pytest.mark.parametrize("how", ["equal_kernels", "equal_choices", "zero_power", "zero_comm",
                                 "quantised"])
def test_pruned_ties(oracle_lib, how):
    sp = I.Space(3, 10, 2, 11, (4, 8, 12, 16), (1005.0, 1400.0, 1980.0))
    tab = I.make_tables(sp, seed=9, comm_bytes=(8e6, 2e8))
    if how == "equal_kernels":
        for k in ("t", "pw"):
            tab[k][:] = tab[k][:, :, :1]
    elif how == "equal_choices":
        for k in ("t", "pw"):
            tab[k][..., 1:] = tab[k][..., 1:2]
        for k in ("tc", "pc"):
            tab[k][:] = tab[k][..., :1]
    elif how == "zero_power":
        sp = I.Space(3, 10, 2, 11, (4, 8, 12, 16), (1005.0, 1400.0, 1980.0), p_static=0.0)
        tab["pw"][:] = 0.0
        tab["pc"][:] = 0.0
    elif how == "zero_comm":
        tab["tc"][:] = 0.0
    else:
        for k in tab:
            q = np.abs(tab[k]).max() / 8
            tab[k] = np.ceil(tab[k] / q) * q
    _check(oracle_lib, sp, tab)


@pytest.mark.parametrize("pos", [2, 11, 24])
@pytest.mark.parametrize("how", ["line", "ties"])
def test_gathered_candidates(oracle_lib, how, pos):
    """Candidates gather 64 to a frontier: slabs where none beats another (64 time-energy
    trade-offs per launch position on one line, or equal energies throughout) fill the room,
    overflow it and leave more frontiers than one."""
    N = pos - 1
    sp = I.Space(2, N, 2, pos, tuple(range(4, 12)), (1005.0, 1400.0), p_static=0.0)
    tab = I.make_tables(sp, seed=3, comm_bytes=(8e6, 2e8))
    tab["pw"][:] = 0.0
    tab["pc"][:] = 0.0
    if how == "line":
        tab["t"][:] = 1e-3 * np.arange(1, N + 1)[:, None]
        tab["tc"][:, :, 0] = 1.0 + np.arange(8) / 8
        tab["tc"][:, :, 1] = 1.0 + np.arange(8) / 64
        tab["pc"][:] = (3.0 - tab["tc"]) / tab["tc"]
    _check(oracle_lib, sp, tab)
