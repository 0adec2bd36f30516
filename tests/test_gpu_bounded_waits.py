"""Blocks that place their output behind other blocks' wait a bounded time: with no polls
allowed a call returns and reports KR_EHIP or, where every count was there at the first look,
the right result; the next call with the usual bound is whole."""

import numpy as np
import pytest

from paper_2601_17654_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [3000, 65536, 200001])
def test_staircase_gives_up(oracle_lib, monkeypatch, bins):
    import torch

    from paper_2601_17654_amd import binding as kr

    off, T, E = I.compose_frontiers(seed=1, n_parts=8, n_min=50, n_max=300)
    d = [torch.from_numpy(x).cuda() for x in (off, T, E)]
    ref = oracle_lib.compose(off, T, E, bins)
    rb, rlo, rE = oracle_lib.staircase(ref.F, ref.delta, ref.tmin_sum)
    for polls in ("0", None):
        if polls is None:
            monkeypatch.delenv("KR_TEST_WAIT_POLLS")
        else:
            monkeypatch.setenv("KR_TEST_WAIT_POLLS", polls)
        for _ in range(4):
            comp = kr.compose_frontiers(*d, bins)
            status = int(comp.status.item())
            assert np.array_equal(comp.F.cpu().numpy(), ref.F)
            if polls == "0" and status == kr.KR_EHIP:
                continue
            assert status == kr.KR_OK
            sb, slo, sE = comp.staircase()
            assert np.array_equal(sb.cpu().numpy(), rb)
            assert np.array_equal(slo.cpu().numpy(), rlo) and np.array_equal(sE.cpu().numpy(), rE)


def _curve(rng, n):  # every point on the frontier
    p = rng.permutation(n)
    return np.sort(rng.uniform(1, 2, n))[p], np.sort(rng.uniform(1, 2, n))[::-1][p]


@pytest.mark.parametrize("lens", [[3000, 20], [9000, 30, 0, 5000], [2500] + [5] * 255],
                         ids=["raw", "chunks", "units"])
def test_merge_gives_up(oracle_lib, monkeypatch, lens):
    """The first segment takes far longer than the second, whose block meets no count."""
    import torch

    from paper_2601_17654_amd import binding as kr

    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    T, E = _curve(np.random.default_rng(3), off[-1])
    d = [torch.from_numpy(x).cuda() for x in (T, E)]
    monkeypatch.setenv("KR_TEST_WAIT_POLLS", "0")
    with pytest.raises(kr.KrError) as err:
        kr.pareto_filter(*d, off)
    assert err.value.status == kr.KR_EHIP
    monkeypatch.delenv("KR_TEST_WAIT_POLLS")
    fr = kr.pareto_filter(*d, off)
    o, idx = fr.off.cpu().numpy(), fr.idx.cpu().numpy()
    for g in range(len(lens)):
        s = slice(off[g], off[g + 1])
        ix = oracle_lib.pareto(T[s], E[s]) if lens[g] else np.zeros(0, np.int64)
        assert np.array_equal(idx[o[g]:o[g + 1]], ix), g


def test_fused_merge_gives_up(oracle_lib, monkeypatch):
    import torch

    from paper_2601_17654_amd import binding as kr

    sp = I.Space(200, 24, 1, 25, (4, 8, 16, 32), tuple(np.linspace(1005.0, 1980.0, 16)))
    tab = I.make_tables(sp, seed=2, comm_bytes=(4e6, 128e6))
    order = ("t", "pw", "tc", "pc")
    d = [torch.from_numpy(tab[k]).cuda() for k in order]
    ref = oracle_lib.evaluate_and_filter(sp, *(tab[k] for k in order))
    off = np.concatenate([[0], np.cumsum([len(r[0]) for r in ref])])
    monkeypatch.setenv("KR_TEST_WAIT_POLLS", "0")
    try:
        assert np.array_equal(kr.evaluate_and_filter(sp, *d).off.cpu().numpy(), off)
    except kr.KrError as e:
        assert e.status == kr.KR_EHIP
    monkeypatch.delenv("KR_TEST_WAIT_POLLS")
    fr = kr.evaluate_and_filter(sp, *d)
    assert np.array_equal(fr.off.cpu().numpy(), off)
    assert np.array_equal(fr.idx.cpu().numpy(), np.concatenate([r[0] for r in ref]))
