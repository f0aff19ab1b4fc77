"""The lag construction at the edges of its split (blocks of 2^11 lags, shorter transforms for
short grids, groups of r cut by the scratch of one filter) against the oracle's inverse DFT,
at the tolerances of the other lag tests (1e-12 of the largest lag, 1e-11 for derivatives),
and independence of the batch: many filters give the same bits as one at a time."""

import numpy as np
import pytest
import torch

from oracle import noise

pytestmark = pytest.mark.gpu

PARAMS = np.array([[1.0, 0.2, 1.7], [0.5, 0.05, 1.0], [1.3, 0.0, 1.5], [0.8, 3.0, 4.0]])


@pytest.mark.parametrize("n_c,L", [(5, 1 << 12), (64, 1 << 20), (2048, 1 << 13), (2049, 1 << 14), (4097, 1 << 15),
                                   (8193, 1 << 16), (16384, 1 << 18), (3, 256)])
def test_lag_split_edges(n_c, L):
    from paper_0906_1775_amd import noise_lags
    prm = torch.from_numpy(PARAMS).cuda()
    got = noise_lags(prm, 50.0, n_c, L).cpu().numpy()
    der = noise_lags(prm, 50.0, n_c, L, deriv=3).cpu().numpy()
    for k, fp in enumerate(PARAMS):
        want = noise.lags(n_c, 50.0, *fp, L=L)
        assert np.max(np.abs(got[k] - want)) <= 1e-12 * np.max(np.abs(want)), k
        want = noise.lag_derivatives(n_c, 50.0, *fp, L=L)["alpha"]
        assert np.max(np.abs(der[k] - want)) <= 1e-11 * max(np.max(np.abs(want)), 1e-300), k


def test_lags_do_not_depend_on_the_batch():
    from paper_0906_1775_amd import noise_lags
    rng = np.random.default_rng(2)
    p = np.stack([rng.uniform(0.5, 2, 40), rng.uniform(0.05, 0.5, 40), rng.uniform(1, 2, 40)], axis=1)
    every = noise_lags(torch.from_numpy(p).cuda(), 200.0, 5000)
    for k in (0, 17, 39):
        one = noise_lags(torch.from_numpy(p[k:k + 1].copy()).cuda(), 200.0, 5000)
        assert torch.equal(one[0], every[k])
