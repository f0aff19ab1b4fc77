"""Which maps the scatter reads pixel-major: with a thousand hits a pixel only the small ones, whose slices
would leave the chip idle (larger ones take up to twice the time so), and the sums of both forms."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pix,sliced", [(1000, False), (8000, False), (30_000, True), (65_000, True)])
@pytest.mark.parametrize("precision,n_rhs", [("mixed", 1), ("fp64", 1)])
def test_layout_of_many_hits(n_pix, sliced, precision, n_rhs):
    from paper_0906_1775_amd import MapMaker
    dev = torch.device("cuda:0")
    n = max(1 << 26, 1100 * n_pix) + 12_345          # more than 256 MiB of TOD and 1024 hits a pixel
    g = torch.Generator(device=dev)
    g.manual_seed(n_pix)
    pix = torch.randint(0, n_pix, (n,), generator=g, device=dev, dtype=torch.int32)
    y = torch.randn((n_rhs, n), generator=g, device=dev, dtype=torch.float32 if precision == "mixed" else torch.float64)
    mm = MapMaker(pix, None, n_pix, 1, np.array([0, n], dtype=np.int64), np.zeros(1, np.int32),
                  filter_lags=np.ones((1, 1)), n_c=1, precision=precision, n_rhs=n_rhs)
    info = mm.info()
    assert info["n_obs"] == n_pix and (info["n_sliced"] > info["n_valid"]) == sliced
    want = torch.zeros(n_pix, dtype=torch.float64, device=dev).index_add_(0, pix.long(), y[0].double())
    got = mm.point(y)[0, :, 0]
    # sums of n / n_pix values of size 1 in any order: n / n_pix roundings of their largest partial sum
    hits = n / n_pix
    assert float((got - want).abs().max()) <= hits * 2.0 ** -53 * 8.0 * hits ** 0.5
