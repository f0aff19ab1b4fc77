"""The filter that looks its windows up in the float32 search direction of mixed-precision iterations, at every
transform length: one iteration from x = 0 without a preconditioner is x = alpha b with alpha = b.b / (p.q), p = b
rounded to float32 and q = H p rounded to float32, and H p is apply_A's, whose bits are those of gather, filter
and scatter one by one.  So alpha follows from apply_A up to the order of two float64 sums (4e3 terms: 1e-13)."""

import numpy as np
import pytest
import torch

from oracle import noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_stokes,n_rhs", [(1, 1), (1, 3), (3, 1), (3, 3)])
@pytest.mark.parametrize("log_nf", range(11, 17))
def test_first_step(log_nf, n_stokes, n_rhs):
    from paper_0906_1775_amd import MapMaker
    n_f = 1 << log_nf
    n_c = min(n_f // 7 | 1, 8191)
    m = n_f - 2 * n_c
    lens = [n_c - 1, 7, m, m + 1, 2 * m + 3]
    iv = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, n_pix = int(iv[-1]), 1234
    rng = np.random.default_rng(log_nf)
    pix = rng.integers(0, n_pix, n).astype(np.int32)
    pix[rng.random(n) < 0.05] = -1
    w = None
    if n_stokes == 3:
        a = rng.uniform(0.0, 2.0 * np.pi, n)
        w = torch.from_numpy(np.stack([np.sin(a), np.cos(a)], axis=1).astype(np.float32)).cuda()
    lags = noise.lags(n_c, 200.0, 1.0, 0.3, 1.6, L=1 << 17)[None]
    mm = MapMaker(torch.from_numpy(pix).cuda(), w, n_pix, n_stokes, iv, np.zeros(len(lens), np.int32), filter_lags=lags,
                  n_c=n_c, n_f=n_f, precision="mixed", precond="none", n_rhs=n_rhs)
    seen = torch.from_numpy(np.bincount(pix[pix >= 0], minlength=n_pix) > 0).cuda()
    b = torch.from_numpy(rng.standard_normal((n_rhs, n_pix, n_stokes))).cuda() * seen[None, :, None]
    x, _ = mm.solve_rhs(b, fixed_iters=1)
    p = b.float().double()
    q = mm.apply_A(p).float().double()
    alpha = (b * b).sum(dim=(1, 2)) / (p * q).sum(dim=(1, 2))
    want = alpha[:, None, None] * p
    assert float((x - want).abs().max()) <= 1e-13 * float(want.abs().max())
