"""Multi-vector products on both sides of the sizes from which the rows of the
staged X are padded, and with rows of X that are gathered a few times only.
Small whole numbers: every sum is exact in FP32, so the results are compared
for equality."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import gpu_csr, to_dev, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


@pytest.mark.parametrize("per_row", [7, 20])
@pytest.mark.parametrize("n", [1500, 114_000, 260_000])
def test_padded_and_unpadded_rows(n, per_row):
    rng = np.random.default_rng(n + per_row)
    r = np.repeat(np.arange(n), per_row).astype(np.int32)
    c = (np.repeat(rng.integers(0, n - per_row, n), per_row) + np.tile(np.arange(per_row), n)).astype(np.int32)
    v = rng.integers(-3, 4, r.size).astype(np.float64)
    A = oracle.csr_from_coo(n, n, r, c, v)
    X = rng.integers(-3, 4, (n, 31)).astype(np.float64)
    want = oracle.spmm_crs(A, X)
    for dtype, ks in ((torch.float64, (6, 9, 13, 15)), (torch.float32, (11, 15, 17, 31))):
        G = gpu_csr(sp, r, c, v, n, n, dtype)
        J, B = sp.jds_from_csr(G), sp.jds_blocked_windowed_from_csr(G, 64, 4096)
        for k in ks:
            Xd = to_dev(X[:, :k].T.copy()).to(dtype).t()
            for f, M in ((sp.spmm_crs, G), (sp.spmm_jds, J), (sp.spmm_jds_blocked, B)):
                assert np.array_equal(to_np(f(M, Xd)).astype(np.float64), want[:, :k]), (f.__name__, dtype, k)
