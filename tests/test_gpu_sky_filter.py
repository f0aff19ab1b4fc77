"""The filter that looks its windows up in the map against gather, filter and scatter one by one:
P^T N^-1 P x must be the same bits, since every sample has the same value in the same precision.
Every transform length with that form, both precisions, excised samples (pixel 0 holds a large
value that must not leak into them), intervals around the window's lengths, 1 and 3 right-hand
sides."""

import numpy as np
import pytest
import torch

from oracle import noise

pytestmark = pytest.mark.gpu
CASES = [("fp64", k) for k in range(11, 16)] + [("mixed", k) for k in range(11, 17)]


@pytest.mark.parametrize("n_stokes,n_rhs", [(1, 1), (1, 3), (3, 1), (3, 3)])
@pytest.mark.parametrize("precision,log_nf", CASES)
def test_operator_is_its_parts(precision, log_nf, n_stokes, n_rhs):
    from paper_0906_1775_amd import MapMaker
    n_f = 1 << log_nf
    n_c = min(n_f // 7 | 1, 8191)
    m = n_f - 2 * n_c
    lens = [1, 2, n_c - 1, n_c + 1, m - 1, m, m + 1, 2 * m + 3, 5]
    iv = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, n_pix = int(iv[-1]), 333
    assert n_rhs * n <= 1 << 20
    rng = np.random.default_rng(log_nf)
    pix = rng.integers(0, n_pix, n).astype(np.int32)
    pix[rng.random(n) < 0.05] = -1
    w = None
    if n_stokes == 3:
        a = rng.uniform(0.0, 2.0 * np.pi, n)
        w = torch.from_numpy(np.stack([np.sin(a), np.cos(a)], axis=1).astype(np.float32)).cuda()
    lags = np.stack([noise.lags(n_c, 200.0, 1.0, 0.3, 1.6, L=1 << 17), noise.lags(n_c, 200.0, 0.7, 0.1, 1.1, L=1 << 17)])
    mm = MapMaker(torch.from_numpy(pix).cuda(), w, n_pix, n_stokes, iv, (np.arange(len(lens)) % 2).astype(np.int32),
                  filter_lags=lags, n_c=n_c, n_f=n_f, precision=precision, n_rhs=n_rhs)
    x = torch.from_numpy(rng.standard_normal((n_rhs, n_pix, n_stokes))).cuda()
    x[:, 0] = 1e6
    y = mm.unpoint(x, dtype=torch.float64 if precision == "fp64" else torch.float32)
    assert not y[:, torch.from_numpy(pix < 0).cuda()].any()
    assert torch.equal(mm.apply_A(x), mm.point(mm.weight(y)))
