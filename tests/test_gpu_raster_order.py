"""Pixels kept by 8 x 8 tiles of a raster that the TOD shows: P, P^T, hits and a solve against the
oracle on cross-scanned maps whose sides are no multiples of a tile, whose rows do not fill the
last tile or the pixel count, with excised samples and unobserved strips; scans that show no
raster (one axis, random pixels) keep working; an index outside the map is refused as before.

Tolerances as for the operators (float64 1e-12 of the largest output) and the solves (1e-10)."""

import numpy as np
import pytest
import torch

import synth
from gpu_helpers import max_rel, oracle_for, plan_for, rel_err
from oracle import pointing

pytestmark = pytest.mark.gpu
L_K = 1 << 12


def _scan(w, n_pix, n, kind, rng):
    h = -(-n_pix // w)
    t = np.arange(n)
    tri = lambda p, m: np.where(p % (2 * m) < m, p % (2 * m), 2 * m - 1 - p % (2 * m))
    if kind == "random":
        pix = rng.integers(0, n_pix, n)
    else:
        half = n // 2 if kind == "cross" else n
        x, y = tri((0.5 * t).astype(int), w), tri((0.5 * t / w * 1.3).astype(int), h)
        vx, vy = tri((0.5 * t / h * 1.3).astype(int), w), tri((0.5 * t).astype(int), h)
        pix = np.where(t < half, y * w + x, vy * w + vx)
    pix = pix.astype(np.int64)
    pix[pix >= n_pix] = -1
    if kind == "cross":
        pix[(pix % w > w // 2) & (pix % w < w // 2 + 5)] = -1      # a strip no sample sees
    pix[rng.random(n) < 0.03] = -1
    return pix.astype(np.int32)


CASES = [(32, 32 * 32, "cross"), (45, 45 * 61, "cross"), (61, 61 * 45 - 17, "cross"), (157, 157 * 157, "cross"),
         (130, 130 * 160 + 3, "cross"), (64, 64 * 64, "rows"), (64, 64 * 64, "random")]


@pytest.mark.parametrize("n_stokes,n_rhs", [(1, 1), (3, 2)])
@pytest.mark.parametrize("w,n_pix,kind", CASES)
def test_operators(w, n_pix, kind, n_stokes, n_rhs):
    rng = np.random.default_rng(n_pix)
    n = max(9000, 12 * n_pix)
    p = synth.make_custom(n_stokes, grid=(8, 8), det_lens=(n,), n_c=20, f_samp=20.0, n_rhs=n_rhs, seed=3)
    p.n_pix, p.pix = n_pix, _scan(w, n_pix, n, kind, rng)
    p.tod = rng.standard_normal((n_rhs, n))
    if n_stokes == 3:
        a = rng.uniform(0.0, 2.0 * np.pi, n)
        p.w = np.stack([np.sin(a), np.cos(a)], axis=1).astype(np.float32)
    o, mm = oracle_for(p, L_K), plan_for(p, lag_dft_len=L_K, precond="jacobi")   # (pixels of one hit have no block)
    assert np.array_equal(mm.hits().cpu().numpy(), pointing.hits(p.pix, n_pix))
    y = torch.from_numpy(p.tod).cuda()
    xm = mm.point(y).cpu().numpy()
    x = rng.standard_normal((n_rhs, n_pix, n_stokes))
    back = mm.unpoint(torch.from_numpy(x).cuda()).cpu().numpy()
    hx = mm.apply_A(torch.from_numpy(x).cuda()).cpu().numpy()
    m, _ = mm.solve(y, fixed_iters=4)
    for r in range(n_rhs):
        xo = o.to_observed(x[r])
        assert max_rel(xm[r], o.to_global(o.apply_At(p.tod[r]))) <= 1e-12
        assert max_rel(back[r], o.apply_A(xo)) <= 1e-12
        assert max_rel(hx[r], o.to_global(o.apply_H(xo))) <= 1e-12
        ref, _ = o.pcg(o.rhs(p.tod[r]), fixed_iters=4, precond="jacobi")
        assert rel_err(m.cpu().numpy()[r], o.to_global(ref)) <= 1e-10


def test_index_outside_the_map_is_refused():
    rng = np.random.default_rng(1)
    p = synth.make_custom(1, grid=(8, 8), det_lens=(60000,), n_c=20, f_samp=20.0, seed=3)
    p.n_pix = 61 * 61
    good = _scan(61, p.n_pix, 60000, "cross", rng)
    for bad in (p.n_pix, p.n_pix + 40, 2**31 - 1, -2):
        p.pix = good.copy()
        p.pix[777] = bad
        with pytest.raises(Exception, match="outside"):
            plan_for(p, lag_dft_len=L_K)
