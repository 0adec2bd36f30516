"""Batch selection over every tile size of the selection kernel, against the oracle: batches
small and large enough for each, scores that rise along the index (every row beats the
threshold), constant scores (ties only), infinities, and passes of 0 and of 64."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _scores(shape, n, rng):
    if shape == "rising":
        return np.arange(3 * n, dtype=np.float64).reshape(3, n) + 1.0
    if shape == "constant":
        return np.zeros((3, n))
    s = rng.uniform(0, 1, (3, n))
    s[:, rng.random(n) < 0.8] = 0.0
    if shape == "infinite":
        s[0, rng.random(n) < 0.3] = np.inf
        s[1, rng.random(n) < 0.9] = -np.inf
        s[2] = -s[2]
    return s


# 256 * 1024 candidates and each doubling of it up to 32 times: 8 .. 128 rows per wave
@pytest.mark.parametrize("n_cand", [[2047, 2049, 1], [300_000, 0, 250_000], [1_200_001, 77],
                                    [2_300_000], [9_000_000, 100_001]], ids=lambda n: str(sum(n)))
@pytest.mark.parametrize("shape", ["sparse", "rising", "constant", "infinite"])
def test_every_tile_size(oracle_lib, n_cand, shape):
    import torch

    from paper_2601_17654_amd import binding as kr

    rng = np.random.default_rng(sum(n_cand))
    off = np.concatenate([[0], np.cumsum(n_cand)]).astype(np.int64)
    s, unc = _scores(shape, off[-1], rng), np.round(rng.uniform(0, 1, off[-1]), 3)
    obs_off = np.arange(len(n_cand) + 1, dtype=np.int64) * 96
    obs = np.concatenate([rng.integers(0, max(n, 1), 96) for n in n_cand]).astype(np.int64)
    sd, ud = torch.from_numpy(s).cuda(), torch.from_numpy(unc).cuda()
    for ks in ((13, 6, 6, 32), (0, 64, 0, 64), (1, 0, 0, 64)):
        got = kr.select_batch(off, sd, ud, obs_off, obs, *ks).lists()
        ref = oracle_lib.select(off, s, unc, obs_off, obs, *ks)
        for g in range(len(n_cand)):
            np.testing.assert_array_equal(got[g], ref[g], err_msg="%s part %d" % (ks, g))
