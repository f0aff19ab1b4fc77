"""The one-launch iteration step of small maps (one workgroup per right-hand side) against the
oracle's PCG, around the sizes where its rows change shape or end: one thread, a wavefront, 1024
pixels, 4096 (temperature) and 2048 (polarisation) pixels and one more, which takes the general
step; a right-hand side that is zero, and so stopped from the start, beside active ones.

Tolerances of the solves: float64 at a fixed iteration count 1e-10, mixed converged to 1e-8 1e-5."""

import numpy as np
import pytest
import torch

import synth
from gpu_helpers import oracle_for, plan_for, rel_err

pytestmark = pytest.mark.gpu
L_K = 1 << 12


def _problem(n_pix, n_stokes):
    n = max(600, 7 * n_pix)
    p = synth.make_custom(n_stokes, grid=(8, 8), det_lens=(n,), n_c=20, f_samp=20.0, n_rhs=3, seed=n_pix)
    rng = np.random.default_rng(n_pix)
    p.n_pix = n_pix
    p.pix = rng.permutation(np.arange(n) % n_pix).astype(np.int32)
    p.tod = rng.standard_normal((3, n))
    p.tod[1] = 0.0
    if n_stokes == 3:
        a = rng.uniform(0.0, 2.0 * np.pi, n)
        p.w = np.stack([np.sin(a), np.cos(a)], axis=1).astype(np.float32)
    return p


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_stokes,n_pix", [(1, 1), (1, 64), (1, 65), (1, 1024), (1, 1025), (1, 4096), (1, 4097),
                                            (3, 1), (3, 1024), (3, 1025), (3, 2048), (3, 2049)])
def test_small_map_solve(n_stokes, n_pix, precision):
    p = _problem(n_pix, n_stokes)
    o, mm = oracle_for(p, L_K), plan_for(p, precision=precision, lag_dft_len=L_K)
    kw = dict(fixed_iters=5) if precision == "fp64" else dict(tol=1e-8, max_iter=200)
    tod = torch.from_numpy(p.tod).cuda()
    for use_graph in (False, True, True):
        m, info = mm.solve(tod, use_graph=use_graph, **kw)
        m = m.cpu().numpy()
        assert not m[1].any() and info["iters"][1] == 0
        for r in (0, 2):
            ref, _ = o.pcg(o.rhs(p.tod[r]), **({"fixed_iters": 5} if precision == "fp64" else {"tol": 1e-12, "max_iter": 400}))
            assert rel_err(m[r], o.to_global(ref)) <= (1e-10 if precision == "fp64" else 1e-5)
