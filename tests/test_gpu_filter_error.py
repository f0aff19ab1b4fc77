"""Rounding error of N^-1 against the plain transform's, at every length and in both precisions.

The yardstick is the same overlap-save scheme by a library's plain real FFT in the same precision
(scipy.fft keeps float32 and float64), against a convolution in extended precision: the filter may not
be further from the exact output than that on red TODs (a random walk under white noise) and offset
ones, where a transform that spreads slow power over its bins would lose, and no more than a tenth
further on white noise, which is the spread of plain transforms of different radices."""

import numpy as np
import pytest
import scipy.fft
import torch

from oracle import noise

pytestmark = pytest.mark.gpu
N = 200_001
CASES = [("mixed", k, 0) for k in range(7, 19)] + [("fp64", k, 0) for k in range(7, 19) if k != 16] + \
        [("mixed", 15, 4), ("mixed", 16, 3), ("fp64", 15, 6)]


def plain(x, f, n_f):
    """Overlap-save in x's own precision."""
    n_c = len(f)
    m = n_f - 2 * n_c
    c = np.zeros(n_f)
    c[:n_c] = f
    c[n_f - n_c + 1:] = f[1:][::-1]
    sym = np.fft.rfft(c).real.astype(x.dtype)
    k = -(-len(x) // m)
    padded = np.zeros(k * m + 2 * n_c, dtype=x.dtype)
    padded[n_c:n_c + len(x)] = x
    w = np.lib.stride_tricks.sliding_window_view(padded, n_f)[::m][:k]
    y = scipy.fft.irfft(scipy.fft.rfft(w, axis=1) * sym, n=n_f, axis=1)
    assert y.dtype == x.dtype
    return y[:, n_c:n_c + m].reshape(-1)[:len(x)]


def exact(x, f):
    n_c, ld = len(f), np.longdouble
    L = 1 << (len(x) + 2 * n_c - 1).bit_length()
    ker = np.concatenate([f[:0:-1], f]).astype(ld)
    y = scipy.fft.irfft(scipy.fft.rfft(x.astype(ld), n=L) * scipy.fft.rfft(ker, n=L), n=L)
    return y[n_c - 1:n_c - 1 + len(x)]


@pytest.mark.parametrize("precision,log_nf,shape", CASES)
def test_error_of_plain_transform(precision, log_nf, shape):
    from paper_0906_1775_amd import MapMaker
    n_f = 1 << log_nf
    n_c = min(n_f // 5, 8192)
    dt = np.float32 if precision == "mixed" else np.float64
    f = noise.lags(n_c, 200.0, 1.0, 0.2, 1.7)
    dev = torch.device("cuda:0")
    mm = MapMaker(torch.zeros(N, dtype=torch.int32, device=dev), None, 1, 1, np.array([0, N], dtype=np.int64),
                  np.zeros(1, dtype=np.int32), filter_lags=f[None], n_c=n_c, n_f=n_f, precision=precision, fft_shape=shape)
    assert mm.info()["n_f"] == n_f and shape in (0, mm.info()["fft_shape"])
    rng = np.random.default_rng(log_nf)
    white = rng.standard_normal(N)
    for kind, x, bound in (("white", white, 1.1), ("red", white + 0.02 * np.cumsum(rng.standard_normal(N)), 1.0),
                           ("offset", white + 1000.0, 1.0)):
        x = x.astype(dt)
        want = exact(x, f)
        got = mm.weight(torch.from_numpy(x[None]).to(dev)).cpu().numpy()[0]
        e = np.linalg.norm((got - want).astype(np.float64))
        e_plain = np.linalg.norm((plain(x, f, n_f) - want).astype(np.float64))
        assert e <= bound * e_plain, (kind, e / e_plain)
