"""The transform length a plan chooses by itself against the oracle's plain convolution and a
forced length, where the choice changes: correlation lengths from a few samples to thousands
(odd ones too) and intervals far shorter, about as long and far longer than the windows.

Tolerances as for the operators, relative to the largest output: float64 1e-12, float32 1e-5."""

import numpy as np
import pytest
import torch

from oracle import noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[3], [700, 1, 1300], [40000, 2500, 9001], [150001]], ids=lambda v: f"{len(v)}x{max(v)}")
@pytest.mark.parametrize("n_c", [2, 33, 257, 737, 1024, 3001, 8190])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_chosen_length(precision, n_c, lens):
    from paper_0906_1775_amd import MapMaker
    iv = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(iv[-1])
    flt = np.zeros(len(lens), dtype=np.int32)
    lags = noise.lags(n_c, 200.0, 1.0, 0.3, 1.6, L=1 << 17)[None]
    y = np.random.default_rng(n_c).standard_normal((1, n)) + 3.0
    want = noise.apply_ninv(y, iv, flt, lags)
    tol = 1e-12 if precision == "fp64" else 1e-5
    dev = torch.device("cuda:0")
    for n_f in (0, 32768):
        mm = MapMaker(torch.zeros(n, dtype=torch.int32, device=dev), None, 1, 1, iv, flt, filter_lags=lags, n_c=n_c,
                      n_f=n_f, precision=precision)
        f = mm.info()["n_f"]
        assert f > 2 * (n_c - 1) and f & (f - 1) == 0 and (not n_f or f == n_f)
        got = mm.weight(torch.from_numpy(y).to(dev)).cpu().numpy()
        assert np.max(np.abs(got - want)) <= tol * np.max(np.abs(want)), n_f
