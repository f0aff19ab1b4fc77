"""Sums over the samples of a column: the pixel-major scatter with 16, 64 or 512 lanes a pixel
and the half-wave-plate block, against the oracle, at hit counts, pixel counts, segment lengths
and angles where a split can go wrong.

Tolerances as for the operators, relative to the largest output: float64 1e-12, mixed 1e-5
(at most 2^13 samples a column, 64 eps sqrt(2^13) and less)."""

import numpy as np
import pytest
import torch

from gpu_helpers import max_rel
from oracle import pointing
from oracle import templates as tm

pytestmark = pytest.mark.gpu


def _plan(pix, w, n_pix, n_stokes, precision, n_rhs=1, templates=None):
    from paper_0906_1775_amd import MapMaker
    n = pix.shape[0]
    d = torch.device("cuda:0")
    return MapMaker(torch.from_numpy(pix).to(d), None if w is None else torch.from_numpy(w).to(d), n_pix, n_stokes,
                    np.array([0, n], dtype=np.int64), np.zeros(1, dtype=np.int32), filter_lags=np.ones((1, 1)), n_c=1,
                    precision=precision, n_rhs=n_rhs, templates=templates)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("n_stokes,n_rhs", [(1, 1), (1, 5), (3, 1), (3, 3)])
@pytest.mark.parametrize("n_pix,hits", [(1, 15), (1, 5000), (3, 63), (9, 64), (65, 65), (37, 257), (7, 1023), (9, 1025),
                                        (3, 4097), (1030, 64), (1030, 137), (2100, 20), (5000, 140)])
def test_scatter_of_few_pixels(n_pix, hits, n_stokes, n_rhs, precision, tol):
    rng = np.random.default_rng(n_pix * hits)
    n = n_pix * hits
    pix = rng.integers(0, n_pix, n).astype(np.int32) if n_pix > 3 else (np.arange(n) // hits).astype(np.int32)
    pix[rng.random(n) < 0.02] = -1          # unpointed samples
    w = None
    if n_stokes == 3:
        a = rng.uniform(0, 2 * np.pi, n)
        w = np.stack([np.sin(a), np.cos(a)], 1).astype(np.float32)
    y = rng.standard_normal((n_rhs, n))
    mm = _plan(pix, w, n_pix, n_stokes, precision, n_rhs)
    got = mm.point(torch.from_numpy(y).cuda()).cpu().numpy().reshape(n_rhs, n_pix, n_stokes)
    rows = pointing.row_weights(pix, w, n_stokes)
    want = np.zeros((n_rhs, n_pix, n_stokes))
    ok = pix >= 0
    for r in range(n_rhs):
        for c in range(n_stokes):
            want[r, :, c] = np.bincount(pix[ok], weights=(rows[:, c] * y[r])[ok], minlength=n_pix)
    assert max_rel(got, want) <= tol


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("n_pix,hits,n_stokes,n_rhs", [(16385, 3, 3, 5), (40000, 50, 1, 3), (40000, 129, 3, 1),
                                                      (70000, 4, 3, 1), (262209, 3, 3, 2), (262209, 49, 1, 1),
                                                      (262209, 97, 1, 1), (32768, 5, 3, 2), (49152, 140, 1, 1)])
def test_scatter_of_many_pixels(n_pix, hits, n_stokes, n_rhs, precision, tol):
    test_scatter_of_few_pixels(n_pix, hits, n_stokes, n_rhs, precision, tol)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("n_rhs", [1, 3])
@pytest.mark.parametrize("lens,scale", [([1], 1.0), ([1, 0, 1, 4096, 5], 3.0), ([4095, 4097], 1e3), ([255, 1023, 1025, 8193], 4e6),
                                        ([3] * 700, 1e20), ([40000], 6.0), ([17000, 0, 0, 17001, 300], 1e38)])
def test_half_wave_plate_block(lens, scale, n_rhs, precision, tol):
    rng = np.random.default_rng(len(lens))
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(seg[-1])
    om = (scale * rng.uniform(-1, 1, n)).astype(np.float32)
    om[0] = 0.0
    mm = _plan(np.zeros(n, dtype=np.int32), None, 1, 1, precision, n_rhs,
               templates=[dict(kind="hwp", omega=torch.from_numpy(om).cuda(), seg_start=seg)])
    ang, tau = om.astype(np.float64), tm.scaled_time(seg, n)
    k = np.arange(1, 9)
    c, s = np.cos(np.outer(ang, k)), np.sin(np.outer(ang, k))
    cols = np.concatenate([c, tau[:, None] * c, s, tau[:, None] * s], axis=1)
    of = np.searchsorted(seg, np.arange(n), side="right") - 1
    y = rng.standard_normal((n_rhs, n))
    x = rng.standard_normal((n_rhs, 1 + 32 * len(lens)))
    got = mm.point(torch.from_numpy(y).cuda()).cpu().numpy()
    want = np.zeros((n_rhs, 1 + 32 * len(lens)))
    back = np.zeros((n_rhs, n))
    for r in range(n_rhs):
        want[r, 0] = y[r].sum()
        amp = np.zeros((len(lens), 32))
        np.add.at(amp, of, cols * y[r][:, None])
        want[r, 1:] = amp.ravel()
        back[r] = x[r, 0] + (cols * x[r, 1:].reshape(-1, 32)[of]).sum(axis=1)
    assert max_rel(got, want) <= tol
    assert max_rel(mm.unpoint(torch.from_numpy(x).cuda()).cpu().numpy(), back) <= tol


@pytest.mark.parametrize("n_blocks", [1, 3, 4, 16])
def test_many_template_blocks(n_blocks):
    rng = np.random.default_rng(n_blocks)
    n, n_pix, R = 5000, 70, 2
    pix = rng.integers(0, n_pix // 2, n).astype(np.int32)            # half of the map unobserved
    sizes = [int(rng.integers(1, 300)) for _ in range(n_blocks)]
    idx = [rng.integers(-1, max(1, m - m // 3), n).astype(np.int32) for m in sizes]   # and a third of the amplitudes
    mm = _plan(pix, None, n_pix, 1, "fp64", R, [dict(kind="onehot", idx=torch.from_numpy(i).cuda(), n_amp=m)
                                                for i, m in zip(idx, sizes)])
    y = rng.standard_normal((R, n))
    x = rng.standard_normal((R, n_pix + sum(sizes)))
    got = mm.point(torch.from_numpy(y).cuda()).cpu().numpy()
    back = mm.unpoint(torch.from_numpy(x).cuda()).cpu().numpy()
    for r in range(R):
        want, off = [np.bincount(pix, weights=y[r], minlength=n_pix)], n_pix
        tod = x[r, :n_pix][pix]
        for i, m in zip(idx, sizes):
            ok = i >= 0
            want.append(np.bincount(i[ok], weights=y[r][ok], minlength=m))
            tod = tod + np.where(ok, x[r, off:off + m][np.where(ok, i, 0)], 0.0)
            off += m
        assert max_rel(got[r], np.concatenate(want)) <= 1e-12
        assert max_rel(back[r], tod) <= 1e-12
