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
