"""The scratch that the library keeps between calls: bounded, and there for the
process's other allocations when they need it."""
import ctypes

import numpy as np
import pytest

from paper_2310_11186_amd import tsgne

pytestmark = pytest.mark.gpu


def test_kept_scratch_is_bounded_and_makes_way(gpu):
    import torch
    n, k = 300_000, 90
    edges = np.random.default_rng(3).integers(0, n, (n, 2)).astype(np.int32)
    rp, col = (torch.from_numpy(a).to(gpu) for a in tsgne.tsgne_csr_from_edges(n, edges))
    krp = torch.empty(n + 1, dtype=torch.int32, device=gpu)
    kcol = torch.empty(2 * n * k, dtype=torch.int32, device=gpu)
    nnz = ctypes.c_int64()

    def call():
        st = tsgne.lib().tsgne_knn_graph(n, col.numel(), rp.data_ptr(), col.data_ptr(), k, krp.data_ptr(),
                                         kcol.data_ptr(), kcol.numel(), ctypes.byref(nnz), None)
        assert st == tsgne.TSGNE_OK
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    free = call()
    kept = before - free
    assert 0 <= kept <= 1 << 30
    assert call() == free                                  # and no more with every call
    most = torch.empty(free + kept // 2, dtype=torch.uint8, device=gpu)
    del most
    torch.cuda.empty_cache()
