"""Device memory of noise_lags: what one call needs by mm_noise_lags_workspace_size, and no more than that
or a few small workspaces' worth, however many filters and however long the frequency grid."""

import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_filters", [1, 8])
@pytest.mark.parametrize("n_c,log_len", [(64, 18), (8192, 20), (8192, 24)])
def test_workspace_of_noise_lags(n_c, log_len, n_filters):
    import paper_0906_1775_amd as mmlib
    lib = mmlib.load()
    n = ctypes.c_size_t(0)
    assert lib.mm_noise_lags_workspace_size(n_c, 1 << log_len, ctypes.byref(n)) == 0
    p = torch.tensor([[1.0, 0.2, 1.7]] * n_filters, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    out = mmlib.noise_lags(p, 200.0, n_c, 1 << log_len)
    torch.cuda.synchronize()
    peak = torch.cuda.max_memory_allocated() - before - out.numel() * 8
    assert peak <= max(n.value, 68 << 20) + (4 << 20)     # (an allocation is rounded up by 2 MiB)
