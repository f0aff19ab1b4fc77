"""Map-shaped buffers of 2^32 entries and more (the largest map beside the largest template block): the copies
between their rows and the plan's vectors, against the sums done by hand on the few entries the TOD touches."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_largest_map_beside_largest_template():
    from paper_0906_1775_amd import MapMaker
    n_pix = n_amp = (1 << 31) - 2
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GiB of device memory")
    dev = torch.device("cuda:0")
    n = 1000
    rng = np.random.default_rng(1)
    pix = rng.choice([0, 1, 5, n_pix // 2, n_pix - 2, n_pix - 1], n).astype(np.int32)
    idx = rng.choice([0, 3, n_amp // 3, n_amp - 1], n).astype(np.int32)
    tmpl = [dict(kind="onehot", idx=torch.from_numpy(idx).to(dev), n_amp=n_amp)]
    mm = MapMaker(torch.from_numpy(pix).to(dev), None, n_pix, 1, np.array([0, n], dtype=np.int64), np.zeros(1, np.int32),
                  filter_lags=np.ones((1, 1)), n_c=1, templates=tmpl)
    y = rng.standard_normal((1, n))
    q = mm.point(torch.from_numpy(y).to(dev)).reshape(-1)
    assert q.shape[0] == n_pix + n_amp
    want = {}
    for t in range(n):
        want[int(pix[t])] = want.get(int(pix[t]), 0.0) + y[0, t]
        want[n_pix + int(idx[t])] = want.get(n_pix + int(idx[t]), 0.0) + y[0, t]
    at = torch.tensor(sorted(want), dtype=torch.int64, device=dev)
    got = q[at].cpu().numpy()
    assert np.max(np.abs(got - np.array([want[k] for k in sorted(want)]))) <= 1e-12
    q[at] = 0.0
    assert not any(bool(torch.any(part)) for part in q.split(1 << 28))
    x = torch.zeros((1, n_pix + n_amp), dtype=torch.float64, device=dev)
    x[0, at] = torch.arange(1.0, len(want) + 1, dtype=torch.float64, device=dev)
    val = {k: i + 1.0 for i, k in enumerate(sorted(want))}
    y = mm.unpoint(x, dtype=torch.float64).cpu().numpy()[0]
    assert np.array_equal(y, np.array([val[int(p)] + val[n_pix + int(i)] for p, i in zip(pix, idx)]))
