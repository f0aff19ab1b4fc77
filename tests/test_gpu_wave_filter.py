"""N^-1 with the wavefront-private overlap-save transforms (2^10 .. 2^15 points) against the
oracle's plain convolution, at the lengths where a window can go wrong: intervals of one
sample, shorter and longer than the band, one sample around a whole number of windows, odd
starts, odd and even n_c, float32 and float64 TODs in either precision.

Tolerances, relative to the largest output: float64 1e-12 and float32 1e-5, the operator
tolerances (rounding of about 2 log2(n_f) levels, 30 eps, with a margin for the cancellation
of the band-limited symbol)."""

import numpy as np
import pytest
import torch

from oracle import noise

pytestmark = pytest.mark.gpu

CASES = [("fp64", k) for k in range(11, 16)] + [("mixed", k) for k in range(11, 17)]


@pytest.mark.parametrize("n_c_kind", ["odd", "even", "small"])
@pytest.mark.parametrize("precision,log_nf", CASES)
def test_weight_at_window_edges(precision, log_nf, n_c_kind):
    from paper_0906_1775_amd import MapMaker
    n_f = 1 << log_nf
    n_c = {"odd": n_f // 5 | 1, "even": min(n_f // 4, 8192), "small": 3}[n_c_kind]   # (the float64 filter of a mixed plan ends at n_c < 2^14)
    m = n_f - 2 * n_c
    lens = [1, 2, max(1, n_c - 1), n_c + 1, m - 1, m, m + 1, 2 * m + 3, 5]
    iv = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(iv[-1])
    flt = (np.arange(len(lens)) % 2).astype(np.int32)
    lags = np.stack([noise.lags(n_c, 200.0, 1.0, 0.3, 1.6, L=1 << 17), noise.lags(n_c, 200.0, 0.7, 0.1, 1.1, L=1 << 17)])
    rng = np.random.default_rng(log_nf)
    y = rng.standard_normal((2, n)) + 3.0
    dev = torch.device("cuda:0")
    mm = MapMaker(torch.zeros(n, dtype=torch.int32, device=dev), None, 1, 1, iv, flt, filter_lags=lags, n_c=n_c,
                  n_f=n_f, precision=precision, n_rhs=2)
    assert mm.info()["n_f"] == n_f
    tol = 1e-12 if precision == "fp64" else 1e-5
    for dt in (torch.float64, torch.float32):
        t = torch.from_numpy(y).to(dev).to(dt)
        want = noise.apply_ninv(t.cpu().numpy().astype(np.float64), iv, flt, lags)
        got = mm.weight(t).cpu().numpy()
        err = np.max(np.abs(got - want)) / np.max(np.abs(want))
        assert err <= (tol if dt == torch.float64 else max(tol, 1e-6)), (dt, err)
